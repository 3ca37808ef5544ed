// Rules that the host applies when it sizes, plans and launches, checked without a GPU (tests/test_host_rules.py builds this
// program and runs one check per test: argv[1] names it).
#include <cstdio>
#include <cstring>

#include "../paper_2604_06832_amd/csrc/plan.h"
#include "../paper_2604_06832_amd/csrc/prefill_tiles.h"
#include "../paper_2604_06832_amd/csrc/stream_sync.h"

using namespace bd;

static int failures = 0;
#define CHECK(cond, ...)                                                                                          \
  do {                                                                                                            \
    if (!(cond)) { std::printf("FAILED line %d: %s: ", __LINE__, #cond); std::printf(__VA_ARGS__); std::puts(""); ++failures; } \
  } while (0)

// Every forward that goes to the decode kernels fits their buffers: blocks, and quadratic steps of up to 32 rows.
static void decode_rows_hold_every_forward() {
  for (int large_m = 0; large_m < 2; ++large_m)
    for (int max_block = 1; max_block <= 64; ++max_block) {
      const int rows = decode_rows(max_block, large_m != 0);
      CHECK(rows >= max_block && rows <= 64, "max_block %d", max_block);
      for (int B = 1; B <= max_block && B <= kQuadMaxB; ++B) {
        const int M = B * (B + 1);
        if (large_m ? M <= kStreamRows : M <= max_block) CHECK(M <= rows, "max_block %d, quadratic step of %d rows, buffers of %d", max_block, M, rows);
      }
    }
}

// The barrier words of a launch: from whatever epoch its context has come to, each barrier of the launch waits until it is
// published and passes then.
static void barrier_words_wait_at_every_epoch() {
  const unsigned far[] = {0u, 1u, 144u, 0x7FFFFFFEu, 0x7FFFFFFFu, 0x80000000u, 0x80000001u, 0xC0000000u, 0xFFFFFF70u, 0xFFFFFFFEu, 0xFFFFFFFFu};
  for (unsigned bar : far)
    for (unsigned xbar : far) {
      unsigned words[SY_WORDS];
      for (int i = 0; i < SY_WORDS; ++i) words[i] = sync_word_at_start(i, 30u, bar, xbar);
      CHECK(words[SY_PACE] == 30u && words[SY_DEAD] == 0u && words[SY_ARRIVE] == 0u && words[SY_CBAR] == 0u, "epoch %u", bar);
      for (int w = 0; w < 4; ++w) CHECK(words[SY_LANDED + w] == 0u && words[SY_CONSUMED + w] == 0u, "epoch %u", bar);
      for (unsigned k = 1; k <= 180u; ++k)
        for (int i : {(int)SY_EPOCH, (int)SY_XEPOCH}) {
          const unsigned target = (i == SY_EPOCH ? bar : xbar) + k;
          CHECK(!counter_reached(words[i], target), "barrier %u of a launch from epoch %u does not wait", k, target - k);
          words[i] = target;
          CHECK(counter_reached(words[i], target), "barrier %u of a launch from epoch %u does not pass", k, target - k);
        }
    }
}

// Down projection: the choice is one that can be launched, for every K, and one that was measured (whole prompts of four-layer models,
// every tile shape and split) within 3 % of the best, for several FFN sizes.
static void down_projection_takes_measured_tiles() {
  for (int KS = 2; KS <= 1024; KS += 2)
    for (int NT : {1, 2, 16, 31, 64, 66, 96, 128})
      for (int MTc : {1, 2, 3, 4, 5, 8, 13, 21, 38, 64, 65, 97, 128, 188, 256, 375, 512}) {
        int SK = 0;
        const int tile = down_plan(KS, NT, MTc, SK);
        CHECK(tile >= 0 && tile < kDownShapes && SK >= 1 && SK <= kPfSplit && KS % (2 * SK) == 0, "K steps %d, row tiles %d, token tiles %d: tile %d, %d splits", KS, NT, MTc, tile, SK);
      }
  struct Measured { int hidden, ffn, rows; struct { int wn, tw, sk; } good[12]; };
  static const Measured list[] = {
    {1024, 2816, 600, {{4, 2, 2}, {1, 3, 1}, {1, 4, 1}}},
    {1024, 2816, 1024, {{4, 2, 2}, {1, 4, 1}}},
    {1024, 2816, 2048, {{4, 2, 1}}},
    {1024, 3072, 600, {{4, 2, 3}, {4, 2, 2}, {1, 3, 1}}},
    {1024, 3072, 1024, {{4, 2, 2}, {1, 4, 1}}},
    {1024, 3072, 4096, {{4, 2, 1}}},
    {2048, 4096, 1024, {{4, 2, 1}, {8, 4, 4}, {8, 2, 2}}},
    {2048, 4096, 8192, {{8, 8, 1}}},
    {2048, 5504, 1024, {{4, 2, 1}, {8, 2, 2}, {8, 3, 2}}},
    {2048, 8192, 3000, {{8, 3, 1}, {8, 8, 2}, {8, 4, 1}, {8, 3, 2}}},
    {2048, 11008, 333, {{4, 2, 2}, {8, 2, 4}, {4, 2, 4}, {1, 3, 1}}},
    {2048, 11008, 1024, {{8, 4, 4}}},
    {2048, 11008, 4096, {{8, 8, 2}, {8, 4, 1}}},
    {2048, 11008, 8192, {{8, 8, 1}}},
    {1536, 8960, 128, {{1, 4, 4}, {1, 2, 2}, {1, 3, 2}}},
    {1536, 8960, 2048, {{8, 4, 2}, {8, 8, 4}}},
  };
  for (const Measured& m : list) {
    int SK = 0;
    const PfDownTile& t = kDownTiles[down_plan(m.ffn / 32, m.hidden / 16, ceil_div(m.rows, 16), SK)];
    bool ok = false;
    for (auto& g : m.good) ok = ok || (g.wn == t.wn && g.tw == t.tw && g.sk == SK);
    CHECK(ok, "hidden %d, FFN %d, %d rows: %dx%d tiles, %d splits", m.hidden, m.ffn, m.rows, t.wn, t.tw, SK);
  }
}

// Norm: the kernel that was measured the faster one, two K splits added (us, workgroup per row against wavefront per row).
static void norm_takes_the_faster_kernel() {
  struct { int hidden, rows; float by_rows, by_waves; } const list[] = {
    {256, 384, 3.11f, 2.99f}, {256, 768, 3.31f, 3.05f}, {512, 192, 3.03f, 3.01f}, {512, 512, 3.40f, 3.14f}, {512, 768, 3.72f, 3.25f},
    {1024, 192, 3.27f, 3.78f}, {1024, 384, 3.79f, 3.89f}, {1024, 640, 4.41f, 4.10f}, {1024, 768, 4.74f, 4.23f},
    {1536, 384, 4.25f, 4.86f}, {1536, 768, 5.54f, 5.32f}, {2048, 128, 3.49f, 5.33f}, {2048, 512, 5.35f, 5.83f}, {2048, 1024, 9.44f, 6.48f}};
  for (auto& m : list)
    CHECK(norm_by_rows(m.hidden, m.rows / 16) == (m.by_rows < m.by_waves), "hidden %d, %d rows", m.hidden, m.rows);
}

// LM head as a pipelined product: only where its 32-bit descriptor and offsets reach the whole matrix.
static void lm_head_product_fits_its_descriptor() {
  for (int H : {64, 256, 1024, 2048})
    for (long long bytes = (1ll << 32) - 64 * H; bytes <= (1ll << 32) + 64 * H; bytes += 32 * H) {
      const int vocab = (int)(bytes / (2 * H));
      CHECK(lm_as_product(vocab, H, 64, false) == (bytes < (1ll << 32)), "vocabulary %d, hidden %d", vocab, H);
    }
  CHECK(lm_as_product(151936, 2048, 64, false) && !lm_as_product(151936, 2048, 64, true) && !lm_as_product(1024, 1056, 64, false), "3B shape, staged, odd k-steps");
  // and only for contexts that have forwards of more than 32 rows
  for (int rows = 1; rows <= 1056; ++rows) CHECK(lm_as_product(151936, 2048, rows, false) == (rows > 32), "%d rows", rows);
}

// Every reason to give up has a text of its own, and a cause goes ahead of the barriers that time out because of it.
static void every_device_error_has_its_text() {
  DevState ok{};
  CHECK(dev_error_text(ok) == nullptr, "usable context");
  const int reasons[][2] = {{DE_OTHER, DE_RAISED}, {DE_OTHER, DE_OTHER_XCD}, {DE_IN_WORKGROUP, DE_RING}, {DE_IN_WORKGROUP, DE_LDS_WAIT}, {DE_XCD_BARRIER, 1}, {DE_CHIP_BARRIER, 1}};
  for (auto& r : reasons) {
    DevState st{}, with{};
    st.error[r[0]] = r[1];
    CHECK(dev_error_text(st) != nullptr, "word %d", r[0]);
    for (auto& q : reasons) {
      DevState other{};
      other.error[q[0]] = q[1];
      if (&q != &r) CHECK(std::strcmp(dev_error_text(st), dev_error_text(other)) != 0, "words %d and %d", r[0], q[0]);
    }
    with.error[DE_CHIP_BARRIER] = 1;
    with.error[r[0]] = r[1];
    CHECK(dev_error_text(with) == dev_error_text(st), "word %d behind a barrier's", r[0]);
  }
}

// The phase trace: no forward of two token tiles of the streaming kernel.
static void trace_leaves_out_two_token_tiles() {
  for (int rows = 1; rows <= 1056; ++rows) {
    CHECK(trace_takes(rows, true) == (rows <= 16 || rows > 32), "%d rows", rows);
    CHECK(trace_takes(rows, false), "%d rows, register ring", rows);
  }
}

// Down phase: a workgroup's row tiles have a flag each, whatever hidden size and FFN the context has.
static void down_phase_flags_hold_every_row_group() {
  int most = 0;
  for (int hidden = 32; hidden <= kMaxKW * kWavesPerWG * 32; hidden += 32)
    for (int ksplit = 1; ksplit <= 256; ksplit *= 2) {      // (what FFNs of up to 524288 need)
      MegaPlan P{};
      P.nwg = 256;
      P.ph[PH_DOWN].N = hidden;
      P.ph[PH_DOWN].ksplit = ksplit;
      for (int g = 0; g < P.nwg / ksplit; ++g) {
        const int tiles = phase_tile0(P, PH_DOWN, g + 1) - phase_tile0(P, PH_DOWN, g);
        CHECK(8 + tiles <= kFlagWords && tiles <= kWGThreads, "hidden %d, %d K splits: %d row tiles", hidden, ksplit, tiles);
        most = tiles > most ? tiles : most;
      }
    }
  CHECK(most == kMaxRowTiles, "%d", most);
}

int main(int argc, char** argv) {
  struct { const char* name; void (*run)(); } checks[] = {{"decode_rows", decode_rows_hold_every_forward}, {"barrier_words", barrier_words_wait_at_every_epoch},
                                                                  {"down_plan", down_projection_takes_measured_tiles}, {"norm", norm_takes_the_faster_kernel},
                                                                  {"lm_product", lm_head_product_fits_its_descriptor}, {"device_errors", every_device_error_has_its_text},
                                                                  {"trace", trace_leaves_out_two_token_tiles},
                                                                  {"down_flags", down_phase_flags_hold_every_row_group}};
  for (auto& c : checks)
    if (argc == 2 && std::strcmp(argv[1], c.name) == 0) {
      c.run();
      std::puts(failures == 0 ? "OK" : "NOT OK");
      return failures != 0;
    }
  std::puts("which check?");
  return 2;
}
