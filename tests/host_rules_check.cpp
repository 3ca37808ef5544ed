// Rules that the host applies when it sizes, plans and launches, checked without a GPU (tests/test_host_rules.py builds this
// program and runs one check per test: argv[1] names it).
#include <cstdio>
#include <cstring>

#include "../paper_2604_06832_amd/csrc/plan.h"

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

int main(int argc, char** argv) {
  struct { const char* name; void (*run)(); } checks[] = {{"decode_rows", decode_rows_hold_every_forward}};
  for (auto& c : checks)
    if (argc == 2 && std::strcmp(argv[1], c.name) == 0) {
      c.run();
      std::puts(failures == 0 ? "OK" : "NOT OK");
      return failures != 0;
    }
  std::puts("which check?");
  return 2;
}
