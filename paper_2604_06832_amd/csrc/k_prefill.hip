// Translation unit of the large-M prefill kernels (prefill.h) and the host sequence that runs one chunk of prompt
// rows through all layers.
#include <cmath>

#include "launch.h"
#include "prefill.h"
#include "prefill_tiles.h"

namespace bd {
namespace {

// The register-staged kernel (32*WN rows x 32*TW tokens per workgroup, BKS k-steps per stage): K of any length, and the
// path of BD_FLAG_PREFILL_STAGED.
template <int PH, int WN, int BKS, int TW>
int launch_pf_gemm(hipStream_t s, PfGemmArgs a, int n_rows) {
  static bool attr_set = false;
  constexpr int lds = pf_gemm_lds<WN, BKS, TW>();
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&pf_gemm_kernel<PH, WN, BKS, TW>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  a.NT = n_rows / 16;
  a.RG = ceil_div(a.NT, 2 * WN);
  a.TG = ceil_div(a.MTc, 2 * TW);
  const int grid = ceil_div(a.RG, 8) * 8 * a.TG;
  hipLaunchKernelGGL((pf_gemm_kernel<PH, WN, BKS, TW>), dim3(grid), dim3(kPfThreads), lds, s, a);
  return check_launch();
}

template <int PH, int WN, int TW, int BKS, int NST, bool ODD = false>
int launch_pf_gemm_pipe(hipStream_t s, PfGemmArgs a) {
  static bool attr_set = false;
  constexpr int lds = pf_gemm_pipe_lds<WN, TW, BKS, NST>();
  static_assert(lds <= 160 * 1024, "LDS of one CU");
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&pf_gemm_pipe_kernel<PH, WN, TW, BKS, NST, ODD>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  if (ODD ? a.SK != 1 || a.KS % 2 != 1 : a.SK < 1 || a.KS % (2 * a.SK) != 0) return BD_E_ARG;   // whole turns of the K loop per split
  a.RG = ceil_div(a.NT, 2 * WN);
  a.TG = ceil_div(a.MTc, 2 * TW);
  const int grid = ceil_div(a.RG, 8) * 8 * a.TG * a.SK;
  hipLaunchKernelGGL((pf_gemm_pipe_kernel<PH, WN, TW, BKS, NST, ODD>), dim3(grid), dim3(kPfThreads), lds, s, a);
  return check_launch();
}

// Tile shapes of the pipelined GEMM: 32*WN rows x 32*TW tokens per workgroup, one workgroup per CU.  A shape's cost is the
// number of rounds of the chip (32 CUs per XCD; a row group and its K splits stay on one XCD) times the time of one
// round, measured on the phase's 3B shape (launches back to back, weights from HBM); the cheapest shape is taken.
// (A round is a fixed part and a part per k-step, so the shapes' order could shift with K.  With both parts measured for every
// shape the choice over chunks of 33 to 1056 rows would differ by 0.3 % of the products' time at hidden 256, 0.03 % from
// hidden 1024 on.  The down projection, whose K is the FFN and may be split, does weigh both: prefill_tiles.h.)
struct PfTile { int wn, tw; float us; };
template <int N>
int pick_tile(const PfTile (&t)[N], int NT, int MTc, int SK) {
  int best = 0;
  float cost = 0.f;
  for (int i = 0; i < N; ++i) {
    const float c = (float)tile_rounds(t[i].wn, t[i].tw, NT, MTc, SK) * t[i].us;
    if (i == 0 || c < cost) { best = i; cost = c; }
  }
  return best;
}

int launch_qkv(hipStream_t s, const PfGemmArgs& a) {
  static constexpr PfTile t[] = {{1, 1, 8.3f}, {1, 2, 9.9f}, {3, 2, 13.8f}, {5, 2, 20.f}, {5, 4, 28.f}, {5, 8, 52.f}, {10, 8, 88.f}};
  switch (pick_tile(t, a.NT, a.MTc, 1)) {
    case 0: return launch_pf_gemm_pipe<PH_QKV, 1, 1, 2, 12>(s, a);
    case 1: return launch_pf_gemm_pipe<PH_QKV, 1, 2, 2, 12>(s, a);
    case 2: return launch_pf_gemm_pipe<PH_QKV, 3, 2, 2, 6>(s, a);
    case 3: return launch_pf_gemm_pipe<PH_QKV, 5, 2, 2, 5>(s, a);
    case 4: return launch_pf_gemm_pipe<PH_QKV, 5, 4, 2, 4>(s, a);
    case 5: return launch_pf_gemm_pipe<PH_QKV, 5, 8, 1, 5>(s, a);
    default: return launch_pf_gemm_pipe<PH_QKV, 10, 8, 1, 4>(s, a);
  }
}
int launch_o(hipStream_t s, const PfGemmArgs& a) {
  if (a.SK > 1) {
    static constexpr PfTile t[] = {{1, 2, 5.8f}, {1, 4, 6.5f}, {2, 4, 8.f}};
    switch (pick_tile(t, a.NT, a.MTc, a.SK)) {
      case 0: return launch_pf_gemm_pipe<PH_O, 1, 2, 2, 12>(s, a);
      case 1: return launch_pf_gemm_pipe<PH_O, 1, 4, 2, 7>(s, a);
      default: return launch_pf_gemm_pipe<PH_O, 2, 4, 2, 6>(s, a);
    }
  }
  static constexpr PfTile t[] = {{4, 1, 12.f}, {4, 2, 16.7f}, {4, 4, 23.f}, {4, 8, 44.f}, {8, 8, 70.f}};
  switch (pick_tile(t, a.NT, a.MTc, 1)) {
    case 0: return launch_pf_gemm_pipe<PH_O, 4, 1, 2, 6>(s, a);
    case 1: return launch_pf_gemm_pipe<PH_O, 4, 2, 2, 6>(s, a);
    case 2: return launch_pf_gemm_pipe<PH_O, 4, 4, 2, 4>(s, a);
    case 3: return launch_pf_gemm_pipe<PH_O, 4, 8, 1, 5>(s, a);
    default: return launch_pf_gemm_pipe<PH_O, 8, 8, 1, 4>(s, a);
  }
}
int launch_gu(hipStream_t s, const PfGemmArgs& a) {
  if (a.KS % 2 != 0) {
    // (hidden an odd multiple of 32; a round's times as below: a stage of one k-step instead of two changes them by under a tenth)
    static constexpr PfTile t[] = {{3, 4, 24.f}, {6, 4, 31.f}, {11, 4, 49.f}, {11, 8, 81.f}};
    switch (pick_tile(t, a.NT, a.MTc, 1)) {
      case 0: return launch_pf_gemm_pipe<PH_GU, 3, 4, 1, 9, true>(s, a);
      case 1: return launch_pf_gemm_pipe<PH_GU, 6, 4, 1, 6, true>(s, a);
      case 2: return launch_pf_gemm_pipe<PH_GU, 11, 4, 1, 5, true>(s, a);
      default: return launch_pf_gemm_pipe<PH_GU, 11, 8, 1, 4, true>(s, a);
    }
  }
  static constexpr PfTile t[] = {{3, 2, 20.5f}, {3, 3, 22.f}, {3, 4, 24.f}, {6, 4, 31.f}, {6, 6, 39.f}, {11, 4, 49.f}, {11, 6, 62.f}, {11, 8, 81.f}};
  switch (pick_tile(t, a.NT, a.MTc, 1)) {
    case 0: return launch_pf_gemm_pipe<PH_GU, 3, 2, 2, 7>(s, a);
    case 1: return launch_pf_gemm_pipe<PH_GU, 3, 3, 2, 6>(s, a);
    case 2: return launch_pf_gemm_pipe<PH_GU, 3, 4, 2, 5>(s, a);
    case 3: return launch_pf_gemm_pipe<PH_GU, 6, 4, 1, 6>(s, a);
    case 4: return launch_pf_gemm_pipe<PH_GU, 6, 6, 1, 5>(s, a);
    case 5: return launch_pf_gemm_pipe<PH_GU, 11, 4, 1, 5>(s, a);
    case 6: return launch_pf_gemm_pipe<PH_GU, 11, 6, 1, 4>(s, a);
    default: return launch_pf_gemm_pipe<PH_GU, 11, 8, 1, 4>(s, a);
  }
}
template <int WN, int TW, int BKS, int NST>
int launch_lm_tile(hipStream_t s, PfGemmArgs a) {
  static bool attr_set = false;
  constexpr int lds = pf_gemm_pipe_lds<WN, TW, BKS, NST>();
  static_assert(lds <= 160 * 1024 && WN >= kPfLmMinTiles, "");
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&pf_gemm_pipe_kernel_lm<WN, TW, BKS, NST>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  a.RG = ceil_div(a.NT, 2 * WN);
  a.TG = ceil_div(a.MTc, 2 * TW);
  hipLaunchKernelGGL((pf_gemm_pipe_kernel_lm<WN, TW, BKS, NST>), dim3(ceil_div(a.RG, 8) * 8 * a.TG), dim3(kPfThreads), lds, s, a);
  return check_launch();
}

int launch_down(hipStream_t s, const PfGemmArgs& a, int tile) {
  switch (tile) {
    case 0: return launch_pf_gemm_pipe<PH_DOWN, 1, 2, 2, 12>(s, a);
    case 1: return launch_pf_gemm_pipe<PH_DOWN, 1, 3, 2, 9>(s, a);
    case 2: return launch_pf_gemm_pipe<PH_DOWN, 1, 4, 2, 7>(s, a);
    case 3: return launch_pf_gemm_pipe<PH_DOWN, 4, 2, 2, 6>(s, a);
    case 4: return launch_pf_gemm_pipe<PH_DOWN, 8, 2, 1, 6>(s, a);
    case 5: return launch_pf_gemm_pipe<PH_DOWN, 8, 3, 1, 6>(s, a);
    case 6: return launch_pf_gemm_pipe<PH_DOWN, 8, 4, 1, 5>(s, a);
    default: return launch_pf_gemm_pipe<PH_DOWN, 8, 8, 1, 4>(s, a);
  }
}

// K splits (at most kPfSplit) that divide n_it pipeline iterations evenly.
int k_split(int n_it) {
  for (int sk = kPfSplit; sk > 1; --sk)
    if (n_it % sk == 0) return sk;
  return 1;
}

template <int D, int JT>
int launch_attn_wide(hipStream_t s, const PfAttnArgs& t) {
  static bool attr_set = false;
  constexpr int lds = pf_attn_wide_lds<D, JT>();
  static_assert(lds <= 160 * 1024, "LDS of one CU");
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&pf_attn_wide_kernel<D, JT>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  hipLaunchKernelGGL((pf_attn_wide_kernel<D, JT>), dim3(t.n_q * ceil_div(t.Mc / 16, JT)), dim3(256), lds, s, t);
  return check_launch();
}

}  // namespace

// One chunk of c.rows rows (prompt rows from prompt row c.off, or the tokens of a decode block) at cache position c.n0:
// all layers, K/V into the cache, no LM head.  The kernels work on whole tiles of 16 rows: the rows that pad the last tile are zero on entry, take part
// in every product and write nothing to the cache.  The device-side length is advanced by the caller.
int launch_prefill_chunk(hipStream_t s, const PfChunk& c) {
  const int rows = c.rows;
  const int MTc = ceil_div(rows, 16);
  const int mc = MTc * 16;
  const DevState* skip = c.skippable ? c.st : nullptr;
  if (c.block) {
    hipLaunchKernelGGL(pf_block_embed_kernel, dim3(rows), dim3(kWGThreads), 0, s, c.x, c.H, c.ids, c.mask,
                       c.seed_tokens, c.seed_mask, c.st, c.skippable, c.mask_id, c.table, c.vocab);
  } else {
    hipLaunchKernelGGL(embed_kernel, dim3(rows), dim3(kWGThreads), 0, s, c.x, c.H, c.embeds, c.n_embed, c.ids, c.off,
                       (const uint8_t*)nullptr, c.mask_id, c.table, c.vocab);
  }
  BD_TRY(check_launch());
  if (mc > rows) {
    hipLaunchKernelGGL(zero_rows_kernel, dim3(mc - rows), dim3(kWGThreads), 0, s, c.x + (size_t)rows * c.H, c.H, skip);
    BD_TRY(check_launch());
  }
  hipLaunchKernelGGL(rope_table_kernel, dim3(mc), dim3(64), 0, s, c.rope, c.st, c.D / 2, c.rope_theta, c.quad_W);
  BD_TRY(check_launch());
  const bool norm_rows = !c.staged && norm_by_rows(c.H, MTc);
  PfGemmArgs g{};
  g.MTc = MTc; g.Mvalid = rows; g.rs = c.rs; g.rope = c.rope; g.x = c.x; g.q = c.q; g.max_kb = c.max_kb; g.n0 = c.n0;
  g.act = c.act; g.H = c.H; g.QD = c.QD; g.KVD = c.KVD; g.D = c.D; g.n_q = c.n_q;
  g.SK = 1;
  g.st = c.st; g.skippable = c.skippable; g.pages = c.pages;
  int parts = 0;                                   // K splits of the last down projection still to be added to x
  auto norm = [&](const float* gain, const float* kparts, int n_kparts) -> int {
    if (norm_rows) hipLaunchKernelGGL(pf_norm_row_kernel, dim3(mc), dim3(kPfThreads), 0, s, c.x, c.H, c.rms_eps, c.xb, MTc, c.rs, gain, kparts, n_kparts, skip);
    else hipLaunchKernelGGL(pf_norm_kernel, dim3(mc / 4), dim3(kPfThreads), 0, s, c.x, c.H, c.rms_eps, c.xb, MTc, c.rs, gain, kparts, n_kparts, skip);
    return check_launch();
  };
  for (int l = 0; l < c.L; ++l) {
    const u16* wl = c.w + (size_t)l * c.layer_elems;
    g.Kc = c.Kc + (size_t)l * c.kv_layer_elems;
    g.Vc = c.Vc + (size_t)l * c.kv_layer_elems;
    // e4m3 weights: the norm gains go into the activation copy and the row scales onto the accumulators (as in decode)
    const float* ws = c.fp8 ? c.wscale + (size_t)l * c.wscale_layer : nullptr;
    BD_TRY(norm(c.fp8 ? c.gains + (size_t)(2 * l) * c.H : nullptr, c.part, parts));
    parts = 0;
    g.w = reinterpret_cast<const bf16x8*>(wl + c.w_off[0]); g.KS = ceil_div(c.H, 32);
    g.xin = reinterpret_cast<const bf16x8*>(c.xb);
    g.wscale = ws ? ws + c.wscale_off[0] : nullptr;
    // (every phase: the pipelined kernel when K is a whole number of its turns, else the register-staged one; gate/up, half
    // of a layer's products, at any K)
    g.NT = c.NQKV / 16;
    if (!c.staged && g.KS % 2 == 0) BD_TRY(launch_qkv(s, g));
    else BD_TRY((launch_pf_gemm<PH_QKV, 2, 2, 2>(s, g, c.NQKV)));
    {
      PfAttnArgs t{};
      t.q = c.q; t.Kc = g.Kc; t.Vc = g.Vc; t.max_kb = c.max_kb; t.n0 = c.n0; t.Mc = mc; t.n_q = c.n_q;
      t.n_kv = c.n_kv; t.scale_log2e = 1.4426950408889634f / std::sqrt((float)c.D); t.out = c.ap; t.MTc = MTc;
      t.mode = c.mode; t.Mvalid = rows; t.st = c.st; t.skippable = c.skippable; t.pages = c.pages;
      const int items = t.n_q * (mc / 16);                    // one item per workgroup, its four wavefronts share the blocks
      const bool quad = c.mode >= 2;
      // (few rows: query tiles of a head share a workgroup, the keys are dealt to kPfAttnChunks workgroups, a second
      // kernel sums the chunks)
      const bool split = MTc <= 4 && !c.staged && c.apart != nullptr;
      // Two query tiles per workgroup halve what comes out of the L2s, and the number of workgroups.  (Tiles of 16 rows, keys before
      // the chunk) -> us for one and for two tiles, 16 heads.  They are faster once the one-tile kernel, of which three workgroups of
      // D = 128 fit a CU, needs another round of the chip: D = 128 (48, 0) 14.1 / 14.2, (56, 0) 18.1 / 16.0, (64, 0) 21.1 / 17.9; D = 64 (48, 0)
      // 10.1 / 10.2, (56, 0) 13.2 / 11.4.  With fewer workgroups they are where the loads bound it, D = 128 from 512 keys on: (16, 512)
      // 8.3 / 10.2, (20, 512) 11.5 / 11.0, (33, 128) 11.9 / 12.8, (33, 512) 17.3 / 16.4, (64, 7168) 151 / 92; D = 64, half the bytes per
      // block: (33, 1024) 14.1 / 14.9, (40, 1024) 15.7 / 15.4, (20, 4096) 25.3 / 22.9, (33, 4096) 31.3 / 31.9.
      const bool loads = c.D == 128 ? c.n0 >= 512 : c.n0 >= 4096 || (c.n0 >= 512 && MTc >= 40);
      const bool wide = !split && !quad && (items > 3 * kCUs || (items >= 320 && loads));
      if (split) {
        t.n_chunks = kPfAttnChunks;
        t.part = c.apart;
        const int grid = t.n_kv * ceil_div(mc / 16, kPfAttnTiles) * (t.n_q / t.n_kv) * kPfAttnChunks;
        if (c.D == 128 && quad) hipLaunchKernelGGL((pf_attn_split_kernel<128, kPfAttnTiles, true>), dim3(grid), dim3(256), 0, s, t);
        else if (c.D == 128) hipLaunchKernelGGL((pf_attn_split_kernel<128, kPfAttnTiles>), dim3(grid), dim3(256), 0, s, t);
        else if (quad) hipLaunchKernelGGL((pf_attn_split_kernel<64, kPfAttnTiles, true>), dim3(grid), dim3(256), 0, s, t);
        else hipLaunchKernelGGL((pf_attn_split_kernel<64, kPfAttnTiles>), dim3(grid), dim3(256), 0, s, t);
        BD_TRY(check_launch());
        if (c.D == 128) hipLaunchKernelGGL((pf_attn_merge_kernel<128, kPfAttnChunks>), dim3(items * 2), dim3(256), 0, s, t);
        else hipLaunchKernelGGL((pf_attn_merge_kernel<64, kPfAttnChunks>), dim3(items), dim3(256), 0, s, t);
      } else if (wide) {
        if (c.D == 128) BD_TRY((launch_attn_wide<128, 2>(s, t)));
        else BD_TRY((launch_attn_wide<64, 2>(s, t)));
      } else if (c.D == 128 && quad) hipLaunchKernelGGL((pf_attn_kernel<128, 4, true>), dim3(items), dim3(256), 0, s, t);
      else if (c.D == 128) hipLaunchKernelGGL((pf_attn_kernel<128, 4>), dim3(items), dim3(256), 0, s, t);
      else if (quad) hipLaunchKernelGGL((pf_attn_kernel<64, 4, true>), dim3(items), dim3(256), 0, s, t);
      else hipLaunchKernelGGL((pf_attn_kernel<64, 4>), dim3(items), dim3(256), 0, s, t);
      BD_TRY(check_launch());
    }
    g.w = reinterpret_cast<const bf16x8*>(wl + c.w_off[1]); g.KS = ceil_div(c.QD, 32);
    g.xin = reinterpret_cast<const bf16x8*>(c.ap);
    g.wscale = ws ? ws + c.wscale_off[1] : nullptr;
    g.NT = c.H / 16;
    int o_parts = 0;
    if (!c.staged && g.KS % 2 == 0) {
      // up to 256 rows K is split over workgroups like in the down projection below, and the norm that follows adds the
      // splits (beyond, the norm would lose what the product gains)
      g.SK = MTc <= 16 ? k_split(g.KS / 2) : 1;
      g.part = g.SK > 1 ? c.part : nullptr;
      BD_TRY(launch_o(s, g));
      o_parts = g.SK > 1 ? g.SK : 0;
      g.SK = 1; g.part = nullptr;
    } else {
      BD_TRY((launch_pf_gemm<PH_O, 2, 4, 2>(s, g, c.H)));
    }
    BD_TRY(norm(c.fp8 ? c.gains + (size_t)(2 * l + 1) * c.H : nullptr, o_parts > 0 ? c.part : nullptr, o_parts));
    g.w = reinterpret_cast<const bf16x8*>(wl + c.w_off[2]); g.KS = ceil_div(c.H, 32);
    g.xin = reinterpret_cast<const bf16x8*>(c.xb);
    g.wscale = ws ? ws + c.wscale_off[2] : nullptr;
    g.NT = 2 * c.F / 16;
    if (!c.staged) BD_TRY(launch_gu(s, g));
    else BD_TRY((launch_pf_gemm<PH_GU, 4, 2, 4>(s, g, 2 * c.F)));
    g.w = reinterpret_cast<const bf16x8*>(wl + c.w_off[3]); g.KS = ceil_div(c.F, 32);
    g.xin = reinterpret_cast<const bf16x8*>(c.act);
    g.wscale = ws ? ws + c.wscale_off[3] : nullptr;
    g.NT = c.H / 16;
    // down: K split over workgroups (2048 output rows are too few tiles for the chip); the next norm adds the splits
    if (!c.staged && g.KS % 2 == 0) {
      const int tile = down_plan(g.KS, g.NT, MTc, g.SK);
      g.part = g.SK > 1 ? c.part : nullptr;
      BD_TRY(launch_down(s, g, tile));
      parts = g.SK > 1 ? g.SK : 0;
      g.SK = 1; g.part = nullptr;
    } else {
      BD_TRY((launch_pf_gemm<PH_DOWN, 2, 4, 2>(s, g, c.H)));
    }
  }
  if (parts > 0 || c.lm) {
    // the last layer's splits: the same kernel completes the residual stream (its other outputs serve the LM head over all rows)
    BD_TRY(norm(nullptr, c.part, parts));
  }
  return BD_OK;
}

// The LM head over the c.rows rows the last chunk left: logits (if asked for), argmax and its softmax probability per row.
int launch_lm_large(hipStream_t s, const PfLm& c) {
  PfGemmArgs g{};
  g.MTc = ceil_div(c.rows, 16); g.Mvalid = c.rows; g.rs = c.rs; g.SK = 1; g.st = c.st; g.skippable = c.skippable;
  g.w = reinterpret_cast<const bf16x8*>(c.w); g.NT = c.vocab / 16; g.KS = c.H / 32;
  g.xin = reinterpret_cast<const bf16x8*>(c.xb);
  g.logits = c.logits; g.stats = c.stats;
  if (g.KS % 2 != 0) return BD_E_ARG;
  static constexpr PfTile t[] = {{3, 2, 20.5f}, {3, 3, 22.f}, {3, 4, 24.f}, {6, 4, 31.f}, {6, 6, 39.f}, {11, 4, 49.f}, {11, 6, 62.f}, {11, 8, 81.f}};   // (gate/up's: the same K)
  const int i = pick_tile(t, g.NT, g.MTc, 1);
  switch (i) {
    case 0: BD_TRY((launch_lm_tile<3, 2, 2, 7>(s, g))); break;
    case 1: BD_TRY((launch_lm_tile<3, 3, 2, 6>(s, g))); break;
    case 2: BD_TRY((launch_lm_tile<3, 4, 2, 5>(s, g))); break;
    case 3: BD_TRY((launch_lm_tile<6, 4, 1, 6>(s, g))); break;
    case 4: BD_TRY((launch_lm_tile<6, 6, 1, 5>(s, g))); break;
    case 5: BD_TRY((launch_lm_tile<11, 4, 1, 5>(s, g))); break;
    case 6: BD_TRY((launch_lm_tile<11, 6, 1, 4>(s, g))); break;
    default: BD_TRY((launch_lm_tile<11, 8, 1, 4>(s, g))); break;
  }
  hipLaunchKernelGGL(pf_lm_fold_kernel, dim3(c.rows), dim3(kPfThreads), 0, s, c.stats, ceil_div(g.NT, 2 * t[i].wn), g.MTc * 16, c.row_cand, c.row_conf,
                     c.skippable ? c.st : nullptr);
  return check_launch();
}

}  // namespace bd
