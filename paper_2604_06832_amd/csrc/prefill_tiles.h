// Which tile shape a product of the large-M kernels takes (host only).
#pragma once
#include "common.h"
#include "plan.h"
#include "prefill_args.h"

namespace bd {

constexpr int kXcds = 8, kXcdCUs = 32, kCUs = kXcds * kXcdCUs;     // (an MI355X in one piece)

// Rounds of the chip that a product of NT row tiles and MTc token tiles takes in tiles of 2 wn x 2 tw: one workgroup per CU; a row
// group and its K splits stay on one XCD.
inline int tile_rounds(int wn, int tw, int NT, int MTc, int SK) {
  return ceil_div(ceil_div(ceil_div(NT, 2 * wn), kXcds) * ceil_div(MTc, 2 * tw) * SK, kXcdCUs);
}

// Down projection: a round of a tile shape takes a fixed part (launch, first loads, epilogue) and a part per k-step, in us; without a
// K split the epilogue adds to the residual stream, with one it stores partial sums.  (One round of the chip each, hidden 2048, 8 to 86
// k-steps a split: profiles/pipelined_gemm_rounds.txt.)
struct PfDownTile { int wn, tw; float fixed1, step1, fixed, step; };
constexpr PfDownTile kDownTiles[] = {{1, 2, 3.9f, 0.082f, 3.4f, 0.104f}, {1, 3, 4.0f, 0.105f, 3.8f, 0.127f}, {1, 4, 4.3f, 0.130f, 4.1f, 0.141f},
                                     {4, 2, 5.8f, 0.169f, 5.4f, 0.190f}, {8, 2, 8.3f, 0.288f, 6.6f, 0.327f}, {8, 3, 12.6f, 0.352f, 8.1f, 0.398f},
                                     {8, 4, 18.4f, 0.400f, 9.9f, 0.451f}, {8, 8, 25.3f, 0.709f, 19.2f, 0.730f}};
constexpr int kDownShapes = sizeof(kDownTiles) / sizeof(kDownTiles[0]);

// us of the down projection in tile shape i with SK splits of K: rounds times a round, and the next norm reads the partial sums
// (1 KiB a tile; 1024 rows of hidden 2048 with four splits: 11.9 us against 4.7).
inline float down_cost(int i, int KS, int NT, int MTc, int SK) {
  const PfDownTile& t = kDownTiles[i];
  const float round = SK > 1 ? t.fixed + t.step * (float)(KS / SK) : t.fixed1 + t.step1 * (float)KS;
  return (float)tile_rounds(t.wn, t.tw, NT, MTc, SK) * round + (SK > 1 ? (float)SK * (float)NT * (float)MTc * 2.2e-4f : 0.f);
}

// Tile shape and K splits of the down projection (KS even; a split is a whole number of turns of the loop): the cheapest, or a larger tile
// within 3 % of it (a round that is not full runs a little faster than a full one, and large tiles have fewer workgroups in it).
// Whole prompts of four-layer models (hidden 256 to 2048, FFN 688 to 11008, 40 to 8192 rows), every shape and split timed: the choice is 0.1 %
// slower than the best on average and 2.2 % at most.  (One split for all of a model's sizes and costs measured at 86 k-steps, whatever the
// FFN: 2.5 % and 25 %; hidden 1024, FFN 3072, 600 rows 434 us on 256 x 256 tiles and four splits, 354 with this.)
inline int down_plan(int KS, int NT, int MTc, int& SK) {
  float best = 0.f;
  bool any = false;
  for (int sk = 1; sk <= kPfSplit; ++sk)
    for (int i = 0; i < kDownShapes; ++i)
      if (KS % (2 * sk) == 0) {
        const float c = down_cost(i, KS, NT, MTc, sk);
        if (!any || c < best) { best = c; any = true; }
      }
  int tile = 0;
  float cost = 0.f;
  SK = 0;
  for (int i = kDownShapes - 1; i >= 0 && SK == 0; --i)
    for (int sk = 1; sk <= kPfSplit; ++sk) {
      if (KS % (2 * sk) != 0) continue;
      const float c = down_cost(i, KS, NT, MTc, sk);
      if (c <= best * 1.03f && (SK == 0 || c < cost)) { tile = i; cost = c; SK = sk; }
    }
  return tile;
}

// Does a context's LM head of forwards of more than 32 rows run as a pipelined product over a tile-major copy of its weights (3B shape:
// 622 MB)?  Only if it has such forwards (rows_max: its largest).  K must be a whole number of turns of the loop, and descriptor and offsets of
// the product have 32 bits.  (Else the decode path's LM head, as many rows at a time as its buffers hold.)
inline bool lm_as_product(int vocab, int H, int rows_max, bool staged) {
  return rows_max > kStreamRows && !staged && H % 64 == 0 && (size_t)vocab * (size_t)H * 2 < ((size_t)1 << 32);
}

// Norm of a chunk: one workgroup per row while the rows do not fill the chip several times over, beyond that one wavefront per row, which
// passes over a row 512 columns at a time.  The more passes, the longer a row keeps its wavefront, and the further the workgroups reach; with
// one pass they have nothing to win (us, workgroup / wavefront per row, two K splits added: hidden 512 384 rows 3.25 / 3.08; 1024 384 rows
// 3.79 / 3.89, 512 rows 4.09 / 3.98; 1536 512 rows 4.71 / 5.03, 640 rows 5.19 / 5.17; 2048 512 rows 5.35 / 5.83, 640 rows 6.04 / 5.98, with four
// splits 768 rows 8.55 / 9.31; whole prompts of the 3B shape: 600 rows 6005 / 6060, 1024 7290 / 7250).  Up to 128 rows either is within
// 0.1 us or the workgroup is ahead.
inline bool norm_by_rows(int H, int MTc) {
  const int passes = ceil_div(H, 512);
  return MTc <= 8 || (passes > 1 && MTc <= 12 * passes);
}

}  // namespace bd
