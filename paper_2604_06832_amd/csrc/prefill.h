// Large-M prefill (Alg. 1 "prefill": one causal forward over the prompt that fills the KV cache).
//
// The decode kernels stream every weight once per forward of at most 64 rows, so a prompt of n tokens pushed
// through them re-reads the model n/64 times.  For the bulk of the prompt this file provides the compute-bound
// form: chunks of up to 8192 rows, each layer as a sequence of tiled MFMA GEMMs with the same fused epilogues as the
// decode path (RMS factor, rotary + Q store + K/V store; residual add; SwiGLU) and a causal attention kernel that
// walks the packed cache with the decode path's per-block routine.  Blocks and quadratic steps of more than 32 rows go the same
// way, with an LM head over all of their rows (pf_gemm_pipe_kernel_lm); a prompt needs it for its last rows alone, which
// the decode path's LM head takes.
//
// Operand layout: both GEMM operands are kept as 1-KiB MFMA fragments (16 rows x 32 k, lane (row i, k-quarter kq)
// holds 8 consecutive k at lane*16 bytes).  Weights: fragment (row tile T, k-step ks) of a layer's phase at
// ((T*KS + ks)*64 + lane) 16-byte units, rows in the decode path's phase-row order (rotary pairs of q/k adjacent,
// (gate f, up f) adjacent, norm gains folded into the columns).  Activations: the packed order of xp_index().
#pragma once
#include <type_traits>

#include "prefill_args.h"
#include "prefill_attn.h"
#include "stream_fwd.h"

namespace bd {

// Epilogue operands of a workgroup tile, read from LDS (their own counter): a load behind a store waits for that store's
// acknowledgement, because vector memory operations are counted in order, and with the row scales and token factors loaded
// tile by tile between the stores the gate/up epilogue of a 352 x 256 tile took about 40 us, as long as its products.
// [AT * 16] scales of the rows (e4m3 weights), then [BT * 16] token factors 1/rms (QKV, gate/up).
template <int AT, int BT> constexpr int pf_ep_bytes() { return (AT + BT) * 16 * 4; }
template <int PH, int AT, int BT>
__device__ inline void pf_ep_fetch(const PfGemmArgs& a, float* ep, int T0, int mt0) {
  constexpr bool kNorm = PH == PH_QKV || PH == PH_GU || PH == PH_LM;
  for (int i = threadIdx.x; i < AT * 16; i += kPfThreads) ep[i] = a.wscale != nullptr ? a.wscale[min(T0 * 16 + i, a.NT * 16 - 1)] : 1.f;
  if constexpr (kNorm)
    for (int i = threadIdx.x; i < BT * 16; i += kPfThreads) ep[AT * 16 + i] = a.rs[min(mt0 * 16 + i, a.MTc * 16 - 1)];
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // (published by the first barrier of the K loop)
}

__device__ inline uint32_t pack_bf16(float lo, float hi) {
  return (uint32_t)f32_to_bf16_bits(lo) | ((uint32_t)f32_to_bf16_bits(hi) << 16);
}

// Epilogue of both GEMM kernels: lane (token column col, row quad g) of a 16 x 16 accumulator tile holds rows
// r .. r+3 of one token.  The loads that remain (rotary factors, old residual values) precede the stores they go with.
template <int PH, int WN, int TW>
__device__ inline void pf_epilogue(const PfGemmArgs& a, f32x4 (&acc)[WN][TW], const float* ep, char* lds, int T0, int mt0, int wn, int wm,
                                   int lane, int kz = 0) {
  const int col = lane & 15, g = lane >> 4;
  const int Tw = T0 + wn * WN, mtw = mt0 + wm * TW;            // this wavefront's first row tile, first token tile
  const float* ep_rs = ep + 2 * WN * 16 + wm * TW * 16 + col;
  auto scale = [&](int i) { return *reinterpret_cast<const f32x4*>(ep + (wn * WN + i) * 16 + 4 * g); };   // of rows r .. r+3 of tile i
  if constexpr (PH == PH_QKV) {
    // One token tile at a time, the (cos, sin) of the next one's rotary pairs requested ahead of this one's stores.  (All of them up
    // front, 16 bytes per accumulator tile, spill at the largest tiles: 8192 rows on 320 x 256 159 us, in this form 99.)
    const int D = a.D, half = D >> 1;
    int key[TW];
#pragma unroll
    for (int j = 0; j < TW; ++j) key[j] = paged_key(a.pages, a.n0 + min((mtw + j) * 16 + col, a.Mvalid - 1));
    f32x4 cs[2][WN];
    auto fetch = [&](int j, f32x4 (&dst)[WN]) {
      const int tok = min((mtw + j) * 16 + col, a.Mvalid - 1);
#pragma unroll
      for (int i = 0; i < WN; ++i)
        dst[i] = *reinterpret_cast<const f32x4*>(a.rope + (size_t)tok * half + ((((Tw + i) * 16 + 4 * g) % D) >> 1));
    };
    fetch(0, cs[0]);
#pragma unroll
    for (int j = 0; j < TW; ++j) asm volatile("" ::"v"(key[j]));
#pragma unroll
    for (int j = 0; j < TW; ++j) {
      if (j + 1 < TW) fetch(j + 1, cs[(j + 1) & 1]);
#pragma unroll
      for (int i = 0; i < WN; ++i) asm volatile("" ::"v"(cs[j & 1][i]));
      const int token = (mtw + j) * 16 + col;
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        const int r = (Tw + i) * 16 + 4 * g;
        if (Tw + i >= a.NT || token >= a.Mvalid) continue;
        const f32x4 v = acc[i][j] * scale(i) * ep_rs[j * 16], c = cs[j & 1][i];
        if (r < a.QD + a.KVD) {
          // rotary pairs: phase rows (2i, 2i+1) of a head hold dims (i, i + D/2)
          const uint32_t p0 = pack_bf16(v[0] * c[0] - v[1] * c[1], v[1] * c[0] + v[0] * c[1]);
          const uint32_t p1 = pack_bf16(v[2] * c[2] - v[3] * c[3], v[3] * c[2] + v[2] * c[3]);
          u16* dst;
          if (r < a.QD) {
            dst = a.q + (size_t)token * a.n_q * D + r;
          } else {
            const int rk = r - a.QD;
            dst = a.Kc + (size_t)(rk / D) * a.max_kb * 32 * D + kp_index(key[j], rk % D, D / 32);
          }
          *reinterpret_cast<uint64_t*>(dst) = (uint64_t)p0 | ((uint64_t)p1 << 32);
        } else {
          const int rv = r - a.QD - a.KVD;
          u16* vc = a.Vc + (size_t)(rv / D) * a.max_kb * 32 * D + vp_index(key[j], rv % D, D / 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) vc[e * 8] = f32_to_bf16_bits(v[e]);      // (four consecutive dims of one 16-dim tile)
        }
      }
    }
  } else if constexpr (PH == PH_GU) {
    float rs[TW];
#pragma unroll
    for (int j = 0; j < TW; ++j) rs[j] = ep_rs[j * 16];
    // No branches between the tiles: a branch per tile keeps the chains (exponential, division) of different tiles from
    // overlapping.  Tiles past the end store beyond the buffer's range, which drops them.
    const rsrc_t ar = make_rsrc(a.act, (unsigned)((a.NT * 8 + 31) / 32 * a.MTc * 1024));
#pragma unroll
    for (int i = 0; i < WN; ++i) {
      const f32x4 ws = scale(i);
      // rows (2f, 2f+1) = (gate f, up f): a tile's eight features are one 16-byte unit per token, a quarter of it in this lane
      const int off = (((Tw + i) >> 2) * a.MTc + mtw) * 1024 + ((((Tw + i) & 3) * 16 + col) << 4) + 4 * g;
#pragma unroll
      for (int j = 0; j < TW; ++j) {
        const f32x4 v = acc[i][j] * ws * rs[j];
        const uint32_t h = pack_bf16(v[0] / (1.f + __expf(-v[0])) * v[1], v[2] / (1.f + __expf(-v[2])) * v[3]);
        __builtin_amdgcn_raw_buffer_store_b32(h, ar, Tw + i < a.NT && mtw + j < a.MTc ? off + j * 1024 : kOob, 0, 0);
      }
    }
  } else if constexpr (PH == PH_LM) {
    // Logits of four vocabulary entries of a token per lane and tile; the largest one, its id and the sum of exponentials of the
    // workgroup's rows, per token: in the lane, over the four row quads, over the two wavefronts that share the tokens (through
    // the stages of the K loop, which nobody reads any more behind the barrier).
    __syncthreads();
    f32x4* st = reinterpret_cast<f32x4*>(lds);                   // [2 (row half)][2 * TW * 16 tokens]
#pragma unroll
    for (int j = 0; j < TW; ++j) {
      const int token = (mtw + j) * 16 + col;
      const float rs = ep_rs[j * 16];
      float m = -INFINITY, s = 0.f;
      int id = 0x7FFFFFFF;
      f32x4 v[WN];
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        v[i] = acc[i][j] * rs;
        if (Tw + i >= a.NT) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v[i][e] > m || id == 0x7FFFFFFF) { m = v[i][e]; id = (Tw + i) * 16 + 4 * g + e; }   // (ascending ids: equal maxima keep the lower)
      }
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        if (Tw + i >= a.NT) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) s += __expf(v[i][e] - m);
        if (a.logits != nullptr && token < a.Mvalid)
          *reinterpret_cast<f32x4*>(a.logits + (size_t)token * a.NT * 16 + (Tw + i) * 16 + 4 * g) = v[i];
      }
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(m, off);
        const int i2 = __shfl_xor(id, off);
        const float s2 = __shfl_xor(s, off);
        stat_merge(m, id, s, m2, i2, s2);
      }
      if (g == 0) st[wn * (2 * TW * 16) + (wm * TW + j) * 16 + col] = f32x4{m, __int_as_float(id), s, 0.f};
    }
    __syncthreads();
    const int T0g = T0 / (2 * WN), mt0 = mtw - wm * TW;
    for (int t = threadIdx.x; t < 2 * TW * 16 && mt0 * 16 + t < a.MTc * 16; t += kPfThreads) {
      const f32x4 p = st[t], q = st[2 * TW * 16 + t];
      float m = p[0], s = p[2];
      int id = __float_as_int(p[1]);
      stat_merge(m, id, s, q[0], __float_as_int(q[1]), q[2]);
      a.stats[(size_t)T0g * (a.MTc * 16) + mt0 * 16 + t] = f32x4{m, __int_as_float(id), s, 0.f};
    }
  } else if (a.part != nullptr) {
#pragma unroll
    for (int i = 0; i < WN; ++i) {
      if (Tw + i >= a.NT) continue;
#pragma unroll
      for (int j = 0; j < TW; ++j) {
        if (mtw + j >= a.MTc) continue;
        *reinterpret_cast<f32x4*>(a.part + ((size_t)kz * a.MTc * 16 + (mtw + j) * 16 + col) * a.H + (Tw + i) * 16 + 4 * g) = acc[i][j] * scale(i);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TW; ++j) {
      if (mtw + j >= a.MTc) continue;
      float* xp = a.x + (size_t)((mtw + j) * 16 + col) * a.H;
      f32x4 xo[WN];
#pragma unroll
      for (int i = 0; i < WN; ++i) xo[i] = *reinterpret_cast<const f32x4*>(xp + min((Tw + i) * 16, a.NT * 16 - 16) + 4 * g);
#pragma unroll
      for (int i = 0; i < WN; ++i) asm volatile("" ::"v"(xo[i]));
#pragma unroll
      for (int i = 0; i < WN; ++i)
        if (Tw + i < a.NT) *reinterpret_cast<f32x4*>(xp + (Tw + i) * 16 + 4 * g) = xo[i] + acc[i][j] * scale(i);
    }
  }
}

// C[rows of the phase][tokens] = W * X^T, fp32 accumulation, epilogue per phase.  A workgroup computes
// (2*WN*16) rows x (2*TW*16) tokens; each wavefront WN x TW tiles of 16 x 16.  K advances by BKS k-steps per iteration
// through two LDS stages; the operands of a stage travel global memory -> registers -> LDS, the loads of stage i+1
// being issued before the MFMAs of stage i.  (A second register set, two stages ahead, costs more in registers than
// it hides in latency: measured slower for every shape here.)
template <int PH, int WN, int BKS, int TW>
__global__ __launch_bounds__(kPfThreads, (2 * (2 * WN * BKS * 64 + 2 * TW * BKS * 64) * 16 <= 72 * 1024) ? 2 : 1) void pf_gemm_kernel(PfGemmArgs a) {
  constexpr int AT = 2 * WN;                                        // row tiles per workgroup
  constexpr int BT = 2 * TW;                                        // token tiles per workgroup
  constexpr int A_UNITS = AT * BKS * 64, B_UNITS = BT * BKS * 64;   // 16-byte units per stage
  constexpr int STAGE = A_UNITS + B_UNITS;
  constexpr int A_PER = A_UNITS / kPfThreads, B_PER = B_UNITS / kPfThreads;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  bf16x8* sm = reinterpret_cast<bf16x8*>(lds);
  if (a.skippable && a.st->skip) return;
  // Row group rg runs on XCD rg mod 8 for all of its token groups, so that a weight tile is fetched into one L2.
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const int rg = (slot / a.TG) * 8 + xcd, tg = slot % a.TG;
  if (rg >= a.RG) return;
  const int T0 = rg * AT, mt0 = tg * BT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wn = wave >> 1, wm = wave & 1;
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};

  // Operands come through raw buffer loads (an offset past the end returns zeros and moves nothing).  Unit u = thread
  // + 256 i of a stage: for the weights tile u / (BKS*64), unit u mod (BKS*64) of its BKS KiB; for the activations
  // k-step u / 512, unit u mod 512 of the eight token tiles.
  const rsrc_t wr = make_rsrc(a.w, (unsigned)((size_t)a.NT * a.KS * 1024));
  const rsrc_t xr = make_rsrc(a.xin, (unsigned)((size_t)a.KS * a.MTc * 1024));
  struct Regs { bf16x8 a[A_PER], b[B_PER]; };
  constexpr int TU = BKS * 64;                                      // units per weight tile and stage
  const int a_tile = threadIdx.x / TU, a_within = threadIdx.x % TU; // (256 / TU tiles per round of 256 units)
  const int a_base = ((T0 + a_tile) * a.KS) * 1024 + a_within * 16;
  const int a_ksl = a_within >> 6;
  constexpr int UB = BT * 64;                                       // activation units per k-step
  const int b_base = mt0 * 1024 + threadIdx.x * 16;
  const int b_tile = threadIdx.x >> 6;
  auto gload = [&](Regs& R, int it) {
    const int ks0 = it * BKS;
    const bool a_ok = ks0 + a_ksl < a.KS;
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int off = a_base + (i * (kPfThreads / TU) * a.KS + ks0) * 1024;
      R.a[i] = buf_load_b(wr, (a_ok && T0 + a_tile + i * (kPfThreads / TU) < a.NT) ? off : kOob);
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int ksl = (i * kPfThreads) / UB, part = (i * kPfThreads) % UB;      // units part .. part+255 of that k-step
      const int off = b_base + ((ks0 + ksl) * a.MTc) * 1024 + part * 16;
      R.b[i] = buf_load_b(xr, (ks0 + ksl < a.KS && mt0 + b_tile + part / 64 < a.MTc) ? off : kOob);
    }
  };
  auto lstore = [&](const Regs& R, int stage) {
    bf16x8* A = sm + stage * STAGE;
#pragma unroll
    for (int i = 0; i < A_PER; ++i) A[threadIdx.x + i * kPfThreads] = R.a[i];
#pragma unroll
    for (int i = 0; i < B_PER; ++i) A[A_UNITS + threadIdx.x + i * kPfThreads] = R.b[i];
  };

  f32x4 acc[WN][TW];
#pragma unroll
  for (int i = 0; i < WN; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int stage) {
    const bf16x8* A = sm + stage * STAGE;
    const bf16x8* Bm = A + A_UNITS;
#pragma unroll
    for (int ksl = 0; ksl < BKS; ++ksl) {
      bf16x8 af[WN], bfr[TW];
#pragma unroll
      for (int i = 0; i < WN; ++i) af[i] = A[((wn * WN + i) * BKS + ksl) * 64 + lane];
#pragma unroll
      for (int j = 0; j < TW; ++j) bfr[j] = Bm[(ksl * BT + wm * TW + j) * 64 + lane];
#pragma unroll
      for (int i = 0; i < WN; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
  };

  const int n_it = (a.KS + BKS - 1) / BKS;
  float* ep = reinterpret_cast<float*>(lds + 2 * STAGE * 16);
  pf_ep_fetch<PH, AT, BT>(a, ep, T0, mt0);
  Regs R0;
  gload(R0, 0);
  lstore(R0, 0);
  __syncthreads();
  for (int it = 0; it < n_it; ++it) {
    if (it + 1 < n_it) gload(R0, it + 1);
    compute(it & 1);
    if (it + 1 < n_it) lstore(R0, (it + 1) & 1);
    __syncthreads();
  }

  pf_epilogue<PH, WN, TW>(a, acc, ep, lds, T0, mt0, wn, wm, lane);
}

// ---- the same product, pipelined: every phase whose K is a whole number of turns of its loop -----------------------------
// Products and accumulators are named in inline assembly so that the sums are updated in place: from the builtin the compiler
// makes the form with separate source and destination registers, and copies or spills accumulators at the ends of the loop.
// The first 64 tiles of a wavefront sit in accumulation registers, the rest in vector registers.
template <bool ACC>
__device__ inline void mfma_in_place(f32x4& c, const bf16x8& a, const bf16x8& b) {
  if constexpr (ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <bool ACC>
__device__ inline void pin_acc(f32x4& c) {
  if constexpr (ACC) asm volatile("" : "+a"(c));
  else asm volatile("" : "+v"(c));
}
// f(integral constant i) for i = 0 .. N-1, unrolled by construction
template <int N, int I = 0, typename F>
__device__ inline void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

// One workgroup per CU with a tile as large as its registers allow (a wavefront owns up to 512 of them), NST stages of BKS
// k-steps in LDS filled by direct loads, and the LDS reads of the next k-step issued between the products of the current one:
// the fragment of row tile i is read again as soon as the products of row i are issued, those of the tokens go into a
// second register set.  So neither LDS nor barrier is waited for while the matrix cores have work: the K loop of the
// 352 x 256 tile takes 1.02 us per k-step (1.45 PFLOP/s over the chip on random data, 2.1 with zeros in LDS and no loads:
// the clock follows the power), and more stages in flight change nothing.  What is left on top is fixed: launch, first loads and epilogue
// take 16.8 us (gate/up, 352 x 256), 10.0 (down, 256 x 128 x four K splits), 6.9 (QKV, 160 x 64), 5.8 (O, 128 x 64).  Measured on
// the 3B shape (launches back to back) against kernels without the overlap of LDS reads and products (1024 rows: two stages, two
// to four workgroups per CU; 72 rows: two token groups of 64): 1024 rows gate/up 81 us / 98, down 50 / 52, QKV 19.9 / 22.9,
// O 17.1 / 16.7; 72 rows gate/up 20.5 / 33.4, down 15.7 / 25.1, QKV 8.1 / 10.2, O 5.8 / 9.0; 64 rows gate/up 18.9 / 19.7.
// Needs whole turns of the loop per K split (ODD: one k-step more, with stages of one and no split).  With SK > 1 the workgroups of an output tile split K among them and
// each leaves its product in its own slice of `part` (O and down phases), which the norm that follows adds.
template <int PH, int WN, int TW, int BKS, int NST, bool ODD>
__device__ __forceinline__ void pf_gemm_pipe(const PfGemmArgs a) {
  constexpr int AT = 2 * WN, BT = 2 * TW;
  constexpr int AF = AT * BKS, TF = AF + BT * BKS;                  // weight fragments, all fragments of a stage
  constexpr int PER = (TF + 3) / 4;                                 // loads per wavefront and stage
  constexpr int U = 2;                                              // k-steps per turn of the loop
  static_assert(U % BKS == 0 && NST >= 3 && (!ODD || BKS == 1), "");
  static_assert((NST - 2) * PER <= 63, "outstanding loads must fit the counter");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if (a.skippable && a.st->skip) return;
  const int xcd = blockIdx.x % 8, slot0 = blockIdx.x / 8;
  const int per = a.TG * a.SK;
  const int rg = (slot0 / per) * 8 + xcd, tg = (slot0 % per) / a.SK, kz = slot0 % a.SK;
  if (rg >= a.RG) return;
  const int T0 = rg * AT, mt0 = tg * BT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wn = wave >> 1, wm = wave & 1;
  const rsrc_t wr = make_rsrc(a.w, (unsigned)((size_t)a.NT * a.KS * 1024));
  const rsrc_t xr = make_rsrc(a.xin, (unsigned)((size_t)a.KS * a.MTc * 1024));
  const int n_it = a.KS / BKS / a.SK, it0 = kz * n_it;
  // With one token group every workgroup has weights of its own and they all share the activations: the row groups start at
  // different k-steps, so that they do not ask the same channels of the L2 for the same fragment at once (3B gate/up, 96 rows per
  // workgroup, 64 tokens: 18.9 us, all from the first k-step 19.7; 48 tokens 18.5 / 19.2; 128 tokens, 96 x 128 tiles, 23.3 / 24.3).  With several,
  // the workgroups that share weights keep in step (1024 rows, 352 x 256: 81.4 us, from different k-steps 84.6).
  const int rot = a.TG == 1 ? rg * 5 % n_it : 0;

  // Fragment f of a stage: weights (k-step f / AT, row tile f mod AT), then activations (k-step, token tile).  Tiles past
  // the end re-read the last valid one and are dropped by the epilogue; with a fragment count that does not divide by
  // four the last one is loaded more than once (the same bytes to the same place).
  unsigned fo[PER];                                                 // byte offset of this wavefront's fragments at k-step 0
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = min(i * 4 + wave, TF - 1);
    if (f < AF) fo[i] = ((unsigned)min(T0 + f % AT, a.NT - 1) * a.KS + f / AT) * 1024u;
    else fo[i] = ((unsigned)((f - AF) / BT) * a.MTc + min(mt0 + (f - AF) % BT, a.MTc - 1)) * 1024u;
    fo[i] = (unsigned)__builtin_amdgcn_readfirstlane((int)fo[i]);   // (uniform; the loads take it in a scalar register)
  }
  int s_issue = 0, itr = rot;                                       // slot and (rotated) iteration of the next stage to issue
  auto issue = [&]() {
    char* base = lds + s_issue * (TF * 1024);
    const unsigned ka = (unsigned)(it0 + itr) * (BKS * 1024u), kb = ka * (unsigned)a.MTc;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = min(i * 4 + wave, TF - 1);
      if (i * 4 + 3 < AF || (i * 4 < AF && f < AF))
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void_t*)(base + f * 1024), 16, lane * 16, (int)(fo[i] + ka), 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void_t*)(base + f * 1024), 16, lane * 16, (int)(fo[i] + kb), 0, 0);
    }
    s_issue = s_issue + 1 == NST ? 0 : s_issue + 1;
    itr = itr + 1 == n_it ? 0 : itr + 1;
  };

  f32x4 acc[WN][TW];
#pragma unroll
  for (int i = 0; i < WN; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  unrolled<WN>([&](auto i) { unrolled<TW>([&](auto j) { pin_acc<(i * TW + j < 64)>(acc[i][j]); }); });
  bf16x8 af[WN], bf[2][TW];
  const char* fa = lds + (wn * WN) * 1024 + lane * 16;              // this wavefront's first row / token fragment of slot 0
  const char* fb = lds + (AF + wm * TW) * 1024 + lane * 16;

  float* ep = reinterpret_cast<float*>(lds + NST * TF * 1024);
  pf_ep_fetch<PH, AT, BT>(a, ep, T0, mt0);
  for (int it = 0; it < NST - 1 && it < n_it; ++it) issue();
  if (n_it >= NST - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * PER) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < WN; ++i) af[i] = *reinterpret_cast<const bf16x8*>(fa + i * 1024);
#pragma unroll
  for (int j = 0; j < TW; ++j) bf[0][j] = *reinterpret_cast<const bf16x8*>(fb + j * 1024);

  // (The compiler's hazard handling does not look into inline assembly: the build checks that between the two markers
  // nothing but the products touches an accumulator, and nothing but LDS reads writes their operands.)
  asm volatile("; BD_ACC_BEGIN" ::: "memory");
  int it = 0, s_read = 0;                                           // stage of the current k-step, slot of the next one
  const int ksteps = n_it * BKS - (ODD ? 1 : 0);
  for (int k = 0; k < ksteps; k += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ksn = (u + 1) % BKS;                                // the next k-step inside its stage
      if (ksn == 0) {
        // the next k-step opens stage it + 1: its loads are this wavefront's oldest, NST - 3 later stages may stay in flight
        if (it + NST - 1 <= n_it) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 3) * PER) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // (a bare barrier: __syncthreads() is also a fence, which waits for every load in flight and so would empty the
        // pipeline; what a wavefront read from slot it - 1 it has waited for before the products that used it)
        __builtin_amdgcn_s_barrier();
        if (it + NST - 1 < n_it) issue();
        ++it;
        s_read = s_read + 1 == NST ? 0 : s_read + 1;
      }
      const char* na = fa + s_read * (TF * 1024) + ksn * (AT * 1024);   // (behind the last k-step: read and not used)
      const char* nb = fb + s_read * (TF * 1024) + ksn * (BT * 1024);
      __builtin_amdgcn_sched_barrier(0);
      unrolled<WN>([&](auto i) {
#pragma unroll
        for (int j = 0; j < TW; ++j)
          if (j * WN / TW == i) bf[(u + 1) & 1][j] = *reinterpret_cast<const bf16x8*>(nb + j * 1024);
        unrolled<TW>([&](auto j) { mfma_in_place<(i * TW + j < 64)>(acc[i][j], af[i], bf[u & 1][j]); });
        af[i] = *reinterpret_cast<const bf16x8*>(na + i * 1024);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  if constexpr (ODD)                                                // the last k-step: its fragments are in registers by now
    unrolled<WN>([&](auto i) { unrolled<TW>([&](auto j) { mfma_in_place<(i * TW + j < 64)>(acc[i][j], af[i], bf[0][j]); }); });
  asm volatile("s_nop 15\n\ts_nop 15\n\t; BD_ACC_END" ::: "memory");
  unrolled<WN>([&](auto i) { unrolled<TW>([&](auto j) { pin_acc<(i * TW + j < 64)>(acc[i][j]); }); });
  pf_epilogue<PH, WN, TW>(a, acc, ep, lds, T0, mt0, wn, wm, lane, kz);
}
template <int PH, int WN, int TW, int BKS, int NST, bool ODD = false>
__global__ __launch_bounds__(kPfThreads, 1) void pf_gemm_pipe_kernel(PfGemmArgs a) {
  pf_gemm_pipe<PH, WN, TW, BKS, NST, ODD>(a);
}
// LM head over all rows of a large forward, by the same loop: the weights are read once for up to 128 rows, where the decode
// path's LM head takes 64 at a time and, at four token tiles, reads 3.3 TB/s.  3B shape, the fold below included: 64 rows 191 -> 127 us
// (622 MB: 4.9 TB/s), 72 rows 310 -> 128, 210 rows 678 -> 178, 1056 rows 3035 -> 711.
template <int WN, int TW, int BKS, int NST>
__global__ __launch_bounds__(kPfThreads, 1) void pf_gemm_pipe_kernel_lm(PfGemmArgs a) {
  pf_gemm_pipe<PH_LM, WN, TW, BKS, NST, false>(a);
}
// One workgroup per row: the row groups' statistics merged (equal maxima keep the lower id).
__global__ __launch_bounds__(kPfThreads) void pf_lm_fold_kernel(const f32x4* __restrict__ stats, int RG, int stride, int* __restrict__ row_cand,
                                                                float* __restrict__ row_conf, const DevState* st) {
  __shared__ f32x4 part[kPfThreads / 64];
  if (st != nullptr && st->skip) return;
  const int r = blockIdx.x, lane = threadIdx.x & 63;
  float m = -INFINITY, s = 0.f;
  int id = 0x7FFFFFFF;
  for (int p = threadIdx.x; p < RG; p += kPfThreads) {
    const f32x4 v = stats[(size_t)p * stride + r];
    stat_merge(m, id, s, v[0], __float_as_int(v[1]), v[2]);
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const float m2 = __shfl_xor(m, off);
    const int i2 = __shfl_xor(id, off);
    const float s2 = __shfl_xor(s, off);
    stat_merge(m, id, s, m2, i2, s2);
  }
  if (lane == 0) part[threadIdx.x >> 6] = f32x4{m, __int_as_float(id), s, 0.f};
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kPfThreads / 64; ++w) stat_merge(m, id, s, part[w][0], __float_as_int(part[w][1]), part[w][2]);
    row_cand[r] = id;
    row_conf[r] = 1.f / s;
  }
}
template <int WN, int TW, int BKS, int NST> constexpr int pf_gemm_pipe_lds() { return NST * (2 * WN + 2 * TW) * BKS * 1024 + pf_ep_bytes<2 * WN, 2 * TW>(); }

template <int WN, int BKS, int TW> constexpr int pf_gemm_lds() { return 2 * (2 * WN * BKS * 64 + 2 * TW * BKS * 64) * 16 + pf_ep_bytes<2 * WN, 2 * TW>(); }

// ---- block assembly: embedding gather into the fp32 residual stream ---------------------------------
// Row r takes embeds[off + r] while off + r < n_embed, else table[id] with id = ids[off + r - n_embed];
// with a mask array, masked rows take the mask token's embedding instead.
__global__ void embed_kernel(float* __restrict__ x, int H, const float* __restrict__ embeds, int n_embed,
                             const int* __restrict__ ids, int off, const uint8_t* __restrict__ mask,
                             int mask_id, const u16* __restrict__ table, int vocab) {
  const int r = blockIdx.x;
  const int p = off + r;
  if (p < n_embed) {
    for (int c = threadIdx.x; c < H; c += blockDim.x) x[(size_t)r * H + c] = embeds[(size_t)p * H + c];
    return;
  }
  int id = ids[p - n_embed];
  if (mask != nullptr && mask[p - n_embed]) id = mask_id;
  id = min(max(id, 0), vocab - 1);
  for (int c = threadIdx.x; c < H; c += blockDim.x) x[(size_t)r * H + c] = bf16_bits_to_f32(table[(size_t)id * H + c]);
}

// Rows of a decode block into the fp32 residual stream: row r takes the embedding of ids[r], or of the mask token
// where mask[r] is set.  With seed arrays (denoising step), position 0 first takes the carried prediction if it is
// still masked, exactly as the prologue of the decode kernels does.
__global__ void pf_block_embed_kernel(float* __restrict__ x, int H, const int* ids, const uint8_t* mask,
                                      int* seed_tokens, uint8_t* seed_mask, DevState* st,
                                      int skippable, int mask_id, const u16* __restrict__ table, int vocab) {
  __shared__ int s_id;
  const int r = blockIdx.x;
  if (skippable && st->skip) return;
  if (threadIdx.x == 0) {
    if (r == 0 && seed_mask != nullptr) {
      st->seeded = 0;
      if (seed_mask[0]) {
        seed_tokens[0] = st->carry_cand;
        seed_mask[0] = 0;
        st->seeded = 1;
      }
    }
    int id = ids[r];
    if (mask != nullptr && mask[r]) id = mask_id;
    s_id = min(max(id, 0), vocab - 1);
  }
  __syncthreads();
  const int id = s_id;
  for (int c = threadIdx.x; c < H; c += blockDim.x) x[(size_t)r * H + c] = bf16_bits_to_f32(table[(size_t)id * H + c]);
}

// ---- rotary table for positions n .. n+M-1: (cos, sin) of pos * theta^(-2i/d), i < d/2 ------------------
// (quad_W > 0: rows are groups of quad_W tokens, row m sits at position n + m / W + m % W, Alg. 2)
__global__ void rope_table_kernel(float2* __restrict__ tab, const DevState* st, int half, float theta, int quad_W = 0) {
  const int m = blockIdx.x;
  const double pos = (double)(st->n + (quad_W > 0 ? m / quad_W + m % quad_W : m));
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    const double inv = exp2(-log2((double)theta) * (double)i / (double)half);
    const double ang = pos * inv;
    tab[(size_t)m * half + i] = make_float2((float)cos(ang), (float)sin(ang));
  }
}

// One wavefront per row: 1/rms of the fp32 residual row and its bf16 copy in packed order; completes the residual
// row first when the projection before it left its product in K splits (the norm gain lives in
// the weights, the factor is applied by the GEMM epilogue: same arithmetic as the decode path).
__global__ __launch_bounds__(kPfThreads) void pf_norm_kernel(float* __restrict__ x, int H, float eps, u16* __restrict__ xb,
                                                             int MTc, float* __restrict__ rs, const float* __restrict__ gain,
                                                             const float* __restrict__ kparts, int n_kparts,
                                                             const DevState* st = nullptr) {
  if (st != nullptr && st->skip) return;
  // one wavefront per row, four rows per workgroup
  const int token = blockIdx.x * (kPfThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (token >= MTc * 16) return;
  float* row = x + (size_t)token * H;
  float ss = 0.f;
  // eight consecutive columns per lane: two 16-byte loads per source, one 16-byte store of the packed copy
  for (int c = lane * 8; c < H; c += 64 * 8) {
    f32x4 v0 = *reinterpret_cast<const f32x4*>(row + c), v1 = *reinterpret_cast<const f32x4*>(row + c + 4);
    if (n_kparts > 0) {
      // the K splits of the projection before this norm, added in split order
      for (int p = 0; p < n_kparts; ++p) {
        const float* src = kparts + ((size_t)p * MTc * 16 + token) * H + c;
        v0 += *reinterpret_cast<const f32x4*>(src);
        v1 += *reinterpret_cast<const f32x4*>(src + 4);
      }
      *reinterpret_cast<f32x4*>(row + c) = v0;
      *reinterpret_cast<f32x4*>(row + c + 4) = v1;
    }
    union { u16 h[8]; u32x4 q; } o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ss += v0[e] * v0[e] + v1[e] * v1[e];
      o.h[e] = f32_to_bf16_bits(gain != nullptr ? v0[e] * gain[c + e] : v0[e]);
      o.h[4 + e] = f32_to_bf16_bits(gain != nullptr ? v1[e] * gain[c + 4 + e] : v1[e]);
    }
    *reinterpret_cast<u32x4*>(xb + xp_index(token, c, MTc)) = o.q;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if (lane == 0) rs[token] = rsqrtf(ss / (float)H + eps);
}

// The same for shorter chunks (norm_by_rows): one workgroup per row, so that the rows of a 64-row forward spread over 64 CUs
// instead of 16 and every lane has one group of eight columns per pass.  Same sums in the same order per column; the sum
// of squares is reduced over the workgroup's lanes in a fixed order.
__global__ __launch_bounds__(kPfThreads) void pf_norm_row_kernel(float* __restrict__ x, int H, float eps, u16* __restrict__ xb,
                                                                 int MTc, float* __restrict__ rs, const float* __restrict__ gain,
                                                                 const float* __restrict__ kparts, int n_kparts,
                                                                 const DevState* st = nullptr) {
  __shared__ float wsum[kPfThreads / 64];
  if (st != nullptr && st->skip) return;
  const int token = blockIdx.x;
  float* row = x + (size_t)token * H;
  float ss = 0.f;
  for (int c = threadIdx.x * 8; c < H; c += kPfThreads * 8) {
    f32x4 v0 = *reinterpret_cast<const f32x4*>(row + c), v1 = *reinterpret_cast<const f32x4*>(row + c + 4);
    if (n_kparts > 0) {
      for (int p = 0; p < n_kparts; ++p) {
        const float* src = kparts + ((size_t)p * MTc * 16 + token) * H + c;
        v0 += *reinterpret_cast<const f32x4*>(src);
        v1 += *reinterpret_cast<const f32x4*>(src + 4);
      }
      *reinterpret_cast<f32x4*>(row + c) = v0;
      *reinterpret_cast<f32x4*>(row + c + 4) = v1;
    }
    union { u16 h[8]; u32x4 q; } o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ss += v0[e] * v0[e] + v1[e] * v1[e];
      o.h[e] = f32_to_bf16_bits(gain != nullptr ? v0[e] * gain[c + e] : v0[e]);
      o.h[4 + e] = f32_to_bf16_bits(gain != nullptr ? v1[e] * gain[c + 4 + e] : v1[e]);
    }
    *reinterpret_cast<u32x4*>(xb + xp_index(token, c, MTc)) = o.q;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) rs[token] = rsqrtf((wsum[0] + wsum[1] + wsum[2] + wsum[3]) / (float)H + eps);
}

__global__ __launch_bounds__(kPfThreads) void zero_rows_kernel(float* __restrict__ x, int H, const DevState* st = nullptr) {
  if (st != nullptr && st->skip) return;
  for (int c = threadIdx.x; c < H; c += kPfThreads) x[(size_t)blockIdx.x * H + c] = 0.f;
}

}  // namespace bd
