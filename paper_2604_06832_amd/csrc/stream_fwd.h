// The decoder forward as one persistent kernel with DECOUPLED weight streaming (block sizes up to 32).
//
// A block-denoising step at B <= 32 is bound by reading 5.5 GB of layer weights, but its ~180 dependent
// phases each end in a cross-chip hand-over (stores -> acknowledgement -> grid barrier -> loads) during
// which a compute wavefront cannot also keep HBM busy.  So every workgroup (one per compute unit) runs
// two kinds of wavefronts:
//   * four PRODUCERS, one per consumer, that do nothing but copy their consumer's weight stream from HBM
//     into a ring of 1-KiB slots in LDS, by way of registers that hold a further stretch of it.  The
//     stream is the sequence of 16-row x 32-k MFMA A-operand fragments in exactly the order the consumer
//     will multiply them, across all phases and layers, so the producer needs no knowledge of the
//     computation: it runs ahead whenever a slot is free, through barriers and attention phases alike;
//   * four CONSUMERS that hold the activations of their K range in registers, take weight fragments out
//     of the ring, multiply, reduce over the four K ranges through LDS, and run the fused epilogues,
//     the attention phase and the grid barriers.  Their own vector-memory counter only ever tracks the
//     small latency-critical loads and stores of the hand-over, never the bulk stream.
// Producer and consumer talk through two LDS words per ring ("landed", "consumed").  Because the producer
// wavefronts never reach a workgroup barrier, the consumers synchronise among themselves with an LDS
// arrival counter instead of s_barrier.
//
// Weight stream layout, activation buffers, epilogues and the cross-workgroup data discipline (write-once
// buffers, write-through stores, no cache maintenance inside the kernel) are those of mega.h; the two
// kernels are interchangeable on the same context.
#pragma once
#include "attn_plan.h"
#include "mega.h"
#include "stream_sync.h"

namespace bd {

constexpr int kFwdThreads = 512;      // 4 consumer + 4 producer wavefronts
constexpr int kSlots = 24;                  // 1-KiB ring slots per consumer
constexpr int kMirror = 3;                  // copies of the first slots behind the last one: any four fragments in sequence
                                            // are contiguous in LDS, so a group is read with one address
constexpr int kLdsSpin = 1 << 22;           // bound of every LDS wait (a timed-out wait marks the context broken)
constexpr int kRingBytes = (kSlots + kMirror) * 1024;
constexpr int kShareBytes = 40 * 1024;      // K-reduction buffers / attention merge buffers (one region, re-used)
// Sums of squares a lane adds up: one per 16 channels of a row, dealt to 16 lane groups.  (K of the normed phases is not
// split over workgroups, so H is at most what the four K ranges hold.)
constexpr int kSsqPer = kWavesPerWG * kMaxKW * 32 / 16 / 16;
// 16-row tiles a wavefront accumulates before the K ranges are summed
template <int MT> constexpr int round_tiles() { return MT == 1 ? 6 : 4; }

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ inline unsigned lds_addr(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) char*)p;
}
__device__ inline unsigned lds_ld32(unsigned addr) {
  unsigned v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return (unsigned)__builtin_amdgcn_readfirstlane((int)v);
}
// Two words in one round trip.
__device__ inline void lds_ld32_pair(unsigned addr0, unsigned addr1, unsigned& v0, unsigned& v1) {
  unsigned a, b;
  asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(a), "=v"(b) : "v"(addr0), "v"(addr1) : "memory");
  v0 = (unsigned)__builtin_amdgcn_readfirstlane((int)a);
  v1 = (unsigned)__builtin_amdgcn_readfirstlane((int)b);
}
__device__ inline void lds_st32(unsigned addr, unsigned v) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
__device__ inline void lds_inc(unsigned addr) {
  const unsigned one = 1u;
  asm volatile("ds_add_u32 %0, %1" ::"v"(addr), "v"(one) : "memory");
}

// SY_DEAD: what gave up in this workgroup.  kDeadReported: said so itself; else the low bits name the word of DevState::error that the
// consumers set when they leave (a store at the place itself costs the two-tile kernel a spilled register, 32 rows 1997 -> 2014 us).
enum { kDeadReported = 1, kDeadRing = DE_IN_WORKGROUP, kDeadChip = 4 + DE_CHIP_BARRIER };
static_assert(kDeadRing == 2 && kDeadChip == 4 && DE_RING == 2, "words of DevState::error");
struct FwdSync {
  unsigned base;          // LDS address of the synchronisation block
  unsigned cbar_target;   // arrivals expected at the next consumer barrier
  unsigned arrive_target; // arrivals expected at the next grid barrier
  bool dead;              // a wait timed out somewhere in this workgroup: stop waiting, just finish
};

__device__ inline void mark_dead(FwdSync& sy, DevState* st) {
  sy.dead = true;
  lds_st32(sy.base + SY_DEAD * 4, kDeadReported);
  __hip_atomic_store(&st->error[DE_IN_WORKGROUP], DE_LDS_WAIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait until the LDS word at `addr` has reached `target` (wrap-safe); false on time-out or dead workgroup.
__device__ inline bool lds_wait_ge(FwdSync& sy, unsigned addr, unsigned target, DevState* st) {
  if (sy.dead) return false;
  int spins = 0;
  while (!counter_reached(lds_ld32(addr), target)) {
    if ((++spins & 63) == 0) {
      if (lds_ld32(sy.base + SY_DEAD * 4) != 0u) { sy.dead = true; return false; }
      if (spins > kLdsSpin) { mark_dead(sy, st); return false; }
    }
  }
  return true;
}

// Barrier of the four consumer wavefronts.  LDS operations of one wavefront execute in order, so whatever
// a wavefront wrote to LDS before its arrival is visible to the others after theirs.
__device__ inline void cbar(FwdSync& sy, int lane, DevState* st) {
  sy.cbar_target += kWavesPerWG;
  if (lane == 0) lds_inc(sy.base + SY_CBAR * 4);
  lds_wait_ge(sy, sy.base + SY_CBAR * 4, sy.cbar_target, st);
  asm volatile("" ::: "memory");
}

// ---- producer ----------------------------------------------------------------------------------------------
// Row ranges are whole tiles, so a consumer's stream is a plain sequence of 1-KiB fragments: fragment q of the
// forward sits at byte q*1024 of the wavefront's stream, lane l's 16 bytes at l*16.
// The ring alone holds 24 KiB per consumer; the phases that stream almost nothing (QKV, attention, O and their
// hand-overs, a third of a layer's time) would leave HBM idle once it is full.  A producer wavefront owns as many
// registers as a consumer and needs none, so it keeps NS further fragments there: every fragment travels
// HBM -> stash register -> ring slot, the stash being a circular buffer of NS / 4 groups of four fragments between the
// two (fragment f in entry f mod NS).  Filling and draining advance independently: a group is moved to the ring as
// soon as the ring has room (at LDS speed, whatever is in flight), and groups are re-loaded at a bounded rate (a token
// bucket on the 100 MHz clock, its rate a word the consumers write, see StreamPace), so that the deep look-ahead
// never shows up as a deep queue in front of the latency-critical loads of the hand-overs.
// Stash entries are registers and can only be named statically, so the loop sweeps over the groups: at group k it
// moves group k if that is the next to move, then re-loads it if it is the next to load.  The loads are issued from
// inline assembly so that the waits stay in our hands (a compiler-placed wait in front of a conditionally loaded
// register can only be a wait for everything): vector-memory loads return in order, hence the group with y younger
// loads behind it has landed once at most y are outstanding.  The build checks that the compiler keeps the entries in
// place (no copy or spill of a register whose load may still be in flight) between the two markers below.
constexpr int kStash = 48;                       // fragments a producer keeps in registers (4 registers each)
constexpr int kStashGroup = 4;                   // fragments moved or requested per step

// Pace of the requests, in 10-ns ticks per fragment (1 KiB) of a wavefront, by what the consumers are at.  A request in flight
// delays the hand-over beside it (the loads and stores of a CU queue behind each other), a request not made delays a
// later product.  HBM gives every wavefront 1 KiB per 16 ticks when all ask; a layer needs 150 fragments (bf16, 3B shape) in some
// 5200 ticks, 96 of them in gate/up, and ring and stash hold 72.  So the stash is refilled while attention and O run, gate/up and
// down request at a rate HBM can follow, and the requests nearly stop behind the last product of down.  With one rate throughout
// (30 ticks, 10 while at most 24 fragments were buffered) the fast one fell on the down projection's cross-workgroup sum, a chain of
// far round trips, although nothing is urgent between it and the next gate/up (3B shape, 1024 keys: first start to last arrival of the down
// phase 15.2 us a layer at 32 rows; with the rates, 16 rows, 10.1).  The values are the best of a random search over all of them,
// whole forwards timed on the 3B shape, and flat around the optimum (what the search found next to it is within 1 %:
// profiles/streaming_forward_pace_search.txt).  They come from that shape's shares of a layer, not from a rule; the other shapes with this
// attention (hidden 512 to 2048, FFN 1376 to 11008, four layers) are 1 to 8 % faster with them and the barrier below than with one rate.
// One forward before and after: 4 rows 1959 -> 1875 us, 32 rows 2151 -> 2003; e4m3 (half the fragments), 333
// keys, 32 rows 2031 -> 1968.  With e4m3 and one token tile there is so little to request that the one rate stays (1570 us, with a
// rate per phase 1584: the kernel's registers spill over it).
// The rates are those of the attention inside the XCDs.  Where it is split over the chip (LOCAL false: head counts that do not deal out over
// the XCDs, or BD_FLAG_ATTENTION_KEY_SPLIT) attention and barriers take other shares of a layer and one rate is the better one: hidden 1536, 12 heads,
// FFN 8960, eight layers, bf16, 8 keys 1 row 371 -> 353 us and 32 rows 425 -> 392, 700 keys 406 -> 388 and 459 -> 426; e4m3 32 rows 421 -> 411.
struct StreamPace {
  unsigned qkv, attn, o, gu, gu_end, down, down_end;   // from the phase's start; from the last product of gate/up and of down on
  unsigned low, low_ticks;                             // at most `low` fragments requested and not yet consumed: at least this pace
  unsigned burst;                                      // fragments that may be requested back to back
};
template <int MT, bool FP8, bool LOCAL> constexpr bool stream_paced() { return LOCAL && !(FP8 && MT == 1); }
template <int MT, bool FP8, bool LOCAL> constexpr StreamPace stream_pace() {
  if (!stream_paced<MT, FP8, LOCAL>()) return StreamPace{30, 30, 30, 30, 30, 30, 30, 24, 10, 16};
  if (FP8) return StreamPace{70, 40, 24, 22, 40, 11, 120, 16, 14, 8};
  return MT == 1 ? StreamPace{44, 36, 20, 26, 32, 12, 150, 16, 14, 24} : StreamPace{56, 36, 20, 26, 26, 14, 90, 12, 14, 24};
}
static_assert(kStash % kStashGroup == 0 && kSlots % kStashGroup == 0, "whole groups");

__device__ inline unsigned clock_ticks() { return (unsigned)wall_clock64(); }

// The loads that have `younger` loads issued after them have landed once this returns.
__device__ inline void wait_for_loads(unsigned younger) {
  if (younger >= 32u) asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
  else if (younger >= 16u) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (younger >= 8u) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else if (younger >= 4u) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int NS, int MT, bool FP8, bool LOCAL>
__device__ inline void producer_loop_stash(const MegaArgs& a, int cw, char* ring, unsigned sync_base, int lane) {
  constexpr int NG = NS / kStashGroup;
  constexpr StreamPace kPace = stream_pace<MT, FP8, LOCAL>();
  const MegaPlan& P = a.P;
  // (everything the inline assembly takes in scalar registers is made uniform explicitly)
  const unsigned total = (unsigned)__builtin_amdgcn_readfirstlane(a.wtab[blockIdx.x * kWavesPerWG + cw].frags);
  const unsigned total_up = (total + kStashGroup - 1) / kStashGroup * kStashGroup;   // (loads past the end read zeros and move no data)
  const size_t wbase = (size_t)(a.wstream + (size_t)(blockIdx.x * kWavesPerWG + cw) * P.wave_stride);
  const unsigned wlo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)wbase);
  const unsigned whi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(wbase >> 32));
  const rsrc_t wr = make_rsrc(reinterpret_cast<const void*>(((size_t)whi << 32) | wlo), total * 1024u);
  const unsigned landed_addr = sync_base + (SY_LANDED + cw) * 4;
  const unsigned consumed_addr = sync_base + (SY_CONSUMED + cw) * 4;
  const unsigned dead_addr = sync_base + SY_DEAD * 4, pace_addr = sync_base + SY_PACE * 4;
  bf16x8 st[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) st[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
  unsigned issued = 0, moved = 0, consumed = 0;     // fragments (multiples of the group size)
  int fill_g = 0, move_g = 0;                       // stash groups of fragment `issued` / fragment `moved`
  int slot = 0, spins = 0;
  unsigned t_mark = clock_ticks() - kPace.burst * kPace.qkv;   // start with a full bucket
  const bool no_w = __builtin_amdgcn_readfirstlane(a.no_weights) != 0;   // measurement only: everything but the loads
  asm volatile("; BD_STASH_BEGIN" ::: "memory");
  while (moved < total_up) {
    const unsigned now = clock_ticks();
    unsigned pace = kPace.qkv;
    if constexpr (stream_paced<MT, FP8, LOCAL>()) lds_ld32_pair(consumed_addr, pace_addr, consumed, pace);
    else consumed = lds_ld32(consumed_addr);
    const unsigned ticks = issued - consumed <= kPace.low ? min(pace, kPace.low_ticks) : pace;
    unsigned tokens = (now - t_mark) / ticks;
    if (tokens > kPace.burst || no_w) { tokens = kPace.burst; t_mark = now - kPace.burst * ticks; }
    bool progress = false;
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      if (move_g == k && moved < issued) {
        if (moved + kStashGroup - consumed > (unsigned)kSlots) consumed = lds_ld32(consumed_addr);
        if (moved + kStashGroup - consumed <= (unsigned)kSlots) {
          wait_for_loads(issued - moved - kStashGroup);
          bf16x8* dst = reinterpret_cast<bf16x8*>(ring + slot * 1024 + lane * 16);
#pragma unroll
          for (int j = 0; j < kStashGroup; ++j) dst[j * 64] = st[kStashGroup * k + j];
          if (slot == 0) {
#pragma unroll
            for (int j = 0; j < kMirror; ++j) dst[(kSlots + j) * 64] = st[kStashGroup * k + j];
          }
          asm volatile("" ::: "memory");
          moved += kStashGroup;
          lds_st32(landed_addr, min(moved, total));   // LDS executes a wavefront's operations in order
          slot = (slot + kStashGroup == kSlots) ? 0 : slot + kStashGroup;
          move_g = (k + 1 == NG) ? 0 : k + 1;
          progress = true;
        }
      }
      if (fill_g == k && issued < total_up && issued - moved < (unsigned)NS && tokens >= (unsigned)kStashGroup) {
        const int off = (int)(issued * 1024u) + lane * 16;
        if (!no_w) {
#pragma unroll
          for (int j = 0; j < kStashGroup; ++j)
            asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:%3 nt"
                         : "+v"(st[kStashGroup * k + j]) : "v"(off), "s"(wr), "n"(j * 1024) : "memory");
        }
        issued += kStashGroup;
        tokens -= kStashGroup;
        t_mark += kStashGroup * ticks;
        fill_g = (k + 1 == NG) ? 0 : k + 1;
        progress = true;
      }
    }
    if (progress) {
      spins = 0;
    } else {
      __builtin_amdgcn_s_sleep(1);
      if ((++spins & 31) == 0 && (lds_ld32(dead_addr) != 0u || spins > kLdsSpin)) break;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)\n\t; BD_STASH_END" ::: "memory");
}

// Reductions over the four 16-lane rows of a wavefront (the lanes that share a column of a C fragment), with the
// row-swap instructions of gfx950: two VALU operations per step, no LDS traffic.
__device__ inline float rows_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float rows_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// ---- consumer side of the ring -------------------------------------------------------------------------------
struct Ring {
  const char* base;        // this consumer's slots
  unsigned landed_addr, consumed_addr;
  unsigned have;           // fragments known to have landed
  unsigned taken;          // fragments consumed so far
  int slot;
};

// Wait until nf more fragments than were taken have landed.  (Kept small: it is there once per group of fragments.  A
// wait that gives up marks the workgroup dead and makes every later one return at once.)
__device__ inline void ring_need(Ring& rg, FwdSync& sy, int nf) {
  const unsigned need = rg.taken + (unsigned)nf;
  if ((int)(rg.have - need) < 0) {
    int spins = 0;
    do rg.have = lds_ld32(rg.landed_addr);
    while ((int)(rg.have - need) < 0 && ++spins < kLdsSpin);
    if ((int)(rg.have - need) < 0) {
      sy.dead = true;
      lds_st32(sy.base + SY_DEAD * 4, kDeadRing);
      rg.have = need + 0x40000000u;
    }
  }
  asm volatile("" ::: "memory");
}
// Four fragments from slot `slot` on (contiguous: the mirror makes them so).
__device__ inline void ring_read4(const Ring& rg, int slot, u32x4 (&f)[4], int lane) {
  const u32x4* src = reinterpret_cast<const u32x4*>(rg.base + slot * 1024 + lane * 16);
#pragma unroll
  for (int j = 0; j < 4; ++j) f[j] = src[j * 64];
}
// The next nf fragments have been read: hand their slots back (LDS executes a wavefront's operations in order).
__device__ inline void ring_done(Ring& rg, int nf) {
  asm volatile("" ::: "memory");
  rg.taken += (unsigned)nf;
  rg.slot += nf;
  rg.slot -= rg.slot >= kSlots ? kSlots : 0;
  lds_st32(rg.consumed_addr, rg.taken);
}

// e4m3 weights: one ring fragment holds a 16-row tile for TWO k-steps (lane: 8 codes of the even step, then 8 of
// the odd one).  The codes are widened to bf16 in registers (exact) and multiplied with the bf16 MFMA; the
// per-row scale is applied to the accumulators afterwards.
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
__device__ inline void widen_e4m3(const u32x4 raw, bf16x8& even, bf16x8& odd) {
  union { bf16x8 v; bf16x2_t h[4]; } a, b;
  a.h[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[0], 1.0f, false);
  a.h[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[0], 1.0f, true);
  a.h[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[1], 1.0f, false);
  a.h[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[1], 1.0f, true);
  b.h[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2], 1.0f, false);
  b.h[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2], 1.0f, true);
  b.h[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[3], 1.0f, false);
  b.h[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[3], 1.0f, true);
  even = a.v;
  odd = b.v;
}

// One chunk of the stream (one or two 16-row tiles x `steps` fragment steps of one (bf16) or two (e4m3) k-steps) out of
// the ring, four fragments at a time through two register sets: the LDS reads of a group are issued before the MFMAs of
// the group before it, and its slots are handed back at once.  (The last group is read whole: what lies beyond the
// chunk's last fragment is not used.)
template <int MT, bool TWO, bool FP8>
__device__ inline void consume_chunk(Ring& rg, FwdSync& sy, const bf16x8 (&xk)[kMaxKW][MT], int steps, f32x4 (&acc)[kT][MT], int lane) {
  constexpr int KF = FP8 ? 2 : 1;                           // k-steps per fragment
  constexpr int NT = TWO ? 2 : 1, SPG = 4 / NT;             // tiles; fragment steps per group of four
  constexpr int NG = (kMaxKW / KF + SPG - 1) / SPG;
  u32x4 f[2][4];
  auto take = [&](u32x4 (&dst)[4], int nf) {
    ring_need(rg, sy, nf);
    ring_read4(rg, rg.slot, dst, lane);
    ring_done(rg, nf);
    asm volatile("" ::: "memory");                          // the reads are issued before anything that follows
  };
  take(f[0], min(steps * NT, 4));
#pragma unroll
  for (int b = 0; b < NG; ++b) {
    if (b + 1 < NG) {
      asm volatile("" : "+s"(steps));                       // (or every comparison is evaluated up front and kept in registers)
      if ((b + 1) * SPG < steps) take(f[(b + 1) & 1], min((steps - (b + 1) * SPG) * NT, 4));
    }
#pragma unroll
    for (int u = 0; u < SPG; ++u) {
      if (u > 0) {
        asm volatile("" : "+s"(steps));
        if (b * SPG + u >= steps) break;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const u32x4 raw = f[b & 1][u * NT + t];
        if constexpr (FP8) {
          bf16x8 we, wo;
          widen_e4m3(raw, we, wo);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(we, xk[2 * (b * SPG + u)][mt], acc[t][mt], 0, 0, 0);
            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wo, xk[2 * (b * SPG + u) + 1][mt], acc[t][mt], 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw), xk[b * SPG + u][mt], acc[t][mt], 0, 0, 0);
        }
      }
    }
    if (b + 1 < NG) {
      asm volatile("" : "+s"(steps));
      if ((b + 1) * SPG >= steps) break;
    }
  }
}

// What a consumer needs to know of a phase, read from LDS (filled from MegaArgs::wtab when the kernel starts).
struct FwdCtx {
  int layer, n;             // layer index, committed context length
  int pg[3];                // pages of the blocks that hold positions n .. n+63 (the new rows' keys and values)
  f32x4* red;               // LDS [4][kRound * MT][64]: partial tiles of the four K ranges
  float* s_part;            // LDS [4][64] partial sums of squares per consumer
  char* share;              // LDS region shared by the K-reduction and the attention merge
  int* s_flags;             // LDS scratch ints
  const int4* s_plan;       // LDS [4 phases][4 consumers]: WaveTab::ph
};

// ---- epilogues -------------------------------------------------------------------------------------------------
// v: rows r .. r+3 of one token (lane: column = token, row quad).  Every load of an epilogue precedes its first store: a
// load behind a write-through store would have to wait for that store's acknowledgement.
template <int D>
__device__ inline void epilogue_qkv(const MegaArgs& a, const FwdCtx& fc, int token, int r, f32x4 v, f32x4 cs) {
  const MegaPlan& P = a.P;
  const int rel = ((fc.n + token) >> 5) - (fc.n >> 5);      // which of the (at most three) blocks of the new rows
  const int key = ((rel == 0 ? fc.pg[0] : rel == 1 ? fc.pg[1] : fc.pg[2]) << 5) | ((fc.n + token) & 31);   // in its page
  if (r < P.QD + P.KVD) {
    // rotary pairs: phase rows (2i, 2i+1) of a head hold dims (i, i + D/2)
    const uint32_t p0 = (uint32_t)f32_to_bf16_bits(v[0] * cs[0] - v[1] * cs[1]) |
                        ((uint32_t)f32_to_bf16_bits(v[1] * cs[0] + v[0] * cs[1]) << 16);
    const uint32_t p1 = (uint32_t)f32_to_bf16_bits(v[2] * cs[2] - v[3] * cs[3]) |
                        ((uint32_t)f32_to_bf16_bits(v[3] * cs[2] + v[2] * cs[3]) << 16);
    u16* dst;
    if (r < P.QD) {
      dst = a.Q + ((size_t)fc.layer * a.Mp + token) * P.QD + r;
    } else {
      const int rk = r - P.QD;
      dst = a.Kc + (size_t)fc.layer * a.kv_layer_elems + (size_t)(rk / D) * a.max_kb * 32 * D + kp_index(key, rk % D, D / 32);
    }
    st_wt_u64(dst, (uint64_t)p0 | ((uint64_t)p1 << 32));
  } else {
    const int rv = r - P.QD - P.KVD;
    u16* vc = a.Vc + (size_t)fc.layer * a.kv_layer_elems + (size_t)(rv / D) * a.max_kb * 32 * D + vp_index(key, rv % D, D / 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) st_wt_u16(vc + e * 8, f32_to_bf16_bits(v[e]));   // (four consecutive dims of one 16-dim tile)
  }
}

// x_new = x_old + v into residual version `ver`: fp32, bf16 copy (times the next norm's gain with e4m3 weights), sum of
// squares of this tile's 16 channels.
template <bool FP8>
__device__ inline void epilogue_residual(const MegaArgs& a, int ver, int token, int r, f32x4 v, f32x4 xo, f32x4 gn, int g) {
  float ss = 0.f;
  if (token < a.M) {
    const f32x4 o = xo + v;
    st_wt_f32x4(a.xv + ((size_t)ver * a.Mp + token) * a.P.H + r, o);
    ss = o[0] * o[0] + o[1] * o[1] + o[2] * o[2] + o[3] * o[3];
    const f32x4 w = FP8 ? o * gn : o;
    const uint32_t lo = (uint32_t)f32_to_bf16_bits(w[0]) | ((uint32_t)f32_to_bf16_bits(w[1]) << 16);
    const uint32_t hi = (uint32_t)f32_to_bf16_bits(w[2]) | ((uint32_t)f32_to_bf16_bits(w[3]) << 16);
    st_wt_u64(a.xb + (size_t)ver * a.xb_elems + xp_index(token, r, a.MT), (uint64_t)lo | ((uint64_t)hi << 32));
  }
  ss = rows_sum(ss);
  if (g == 0) st_wt_f32(a.ssq + ((size_t)ver * a.ssq_parts + (r >> 4)) * a.Mp + token, ss);
}

// ---- one GEMM phase (consumer wavefronts) ------------------------------------------------------------------------
// The four phases run the same code with the phase as a runtime value: the loads of the activations, the walk over the
// ring and the reduction are there once.  What that is for is the instruction cache (64 KiB for two compute units): every
// hand-over is a chain in which a miss is not hidden by anything.  With a copy per phase, and the partition of the
// rows evaluated in each (64-bit divisions, a fifth of all instructions), the kernel was 156 KB and missed its cache 195,000
// times per forward by the profiler's count; with one copy 70 KB and 4,700
// (and 52 KB with one form of the attention per kernel).  The K ranges are summed once per round of 6 (one token
// tile) or 4 (two: more accumulators spill) row tiles instead of once per pair.  One forward, 3B shape, 1024 keys: 1 row 2116 -> 1995 us,
// 32 rows 2422 -> 2211 us (two token tiles: rounds of 6 tiles 2442, of 2 tiles 2243).
template <int MT, int D, bool FP8, bool LOCAL>
__device__ inline void stream_gemm_phase(const MegaArgs& a, FwdCtx& fc, Ring& rg, FwdSync& sy, int ph, int wave, int lane_in) {
  constexpr int kRound = round_tiles<MT>();
  int lane = lane_in;
  asm volatile("" : "+v"(lane));
  const MegaPlan& P = a.P;
  const int col = lane & 15, g = lane >> 4;
  int row0, n_tiles, w0, KW, KX, ws_off;                     // (KX: k-steps of KW that exist; e4m3 ranges may reach past the end)
  {
    const int4 d = fc.s_plan[ph * kWavesPerWG + wave];
    row0 = __builtin_amdgcn_readfirstlane(d.x);
    const int y = __builtin_amdgcn_readfirstlane(d.y);
    n_tiles = y & 0xFFFF;
    KX = y >> 16;
    w0 = __builtin_amdgcn_readfirstlane(d.z);
    const int w = __builtin_amdgcn_readfirstlane(d.w);
    KW = w & 31;
    ws_off = w >> 5;
  }

#define BD_SUBTS2(k)                                                                                  \
  do {                                                                                                \
    if (a.trace2 != nullptr && fc.layer == 1 && threadIdx.x == 0) a.trace2[(size_t)blockIdx.x * 64 + ph * 12 + (k)] = wall_clock64(); \
  } while (0)
  BD_SUBTS2(0);
  constexpr StreamPace kPace = stream_pace<MT, FP8, LOCAL>();
  if (stream_paced<MT, FP8, LOCAL>() && wave == 0)
    lds_st32(sy.base + SY_PACE * 4, ph == PH_GU ? kPace.gu : ph == PH_DOWN ? kPace.down : ph == PH_O ? kPace.o : kPace.qkv);
  if (n_tiles > 0) {
    const bool norm = ph == PH_QKV || ph == PH_GU;
    const int ver = 2 * fc.layer + (ph == PH_GU ? 1 : 0);
    const u16* src = norm ? a.xb + (size_t)ver * a.xb_elems
                          : (ph == PH_O ? a.ap + (size_t)fc.layer * a.ap_elems : a.act + (size_t)fc.layer * a.act_elems);
    const rsrc_t xr = make_rsrc(src + (size_t)w0 * MT * 512, (unsigned)(KX * MT * 1024));   // (k-steps beyond KX read as zero)
    // this wavefront's share (parts = wave*4 + lane group mod 16) of the sums of squares of every row, ahead of the
    // activations: they are summed while those arrive
    float sv[MT][kSsqPer];
    if (norm) {
      const int parts = ver == 0 ? 1 : P.H >> 4;
      const rsrc_t sr = make_rsrc(a.ssq + (size_t)ver * a.ssq_parts * a.Mp, (unsigned)(parts * a.Mp * 4));
      // (Parts that do not exist read as zero: the whole offset is in the vector offset, the only one the range check covers.
      // How it is formed decides what the compiler keeps in registers: a running offset, pinned, with bf16 weights, 32 rows 2207 us a
      // forward against 2217 with eight sums; the sums with e4m3, 2150 us against 2190.)
      int so = ((wave * 4 + g) * a.Mp + col) * 4;
#pragma unroll
      for (int u = 0; u < kSsqPer; ++u) {
        const int off = so + (FP8 ? u * 16 * a.Mp * 4 : 0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sv[mt][u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, off + mt * 64, 0, 0));
        if constexpr (!FP8) {
          so += 16 * a.Mp * 4;
          asm volatile("" : "+v"(so));
        }
      }
      asm volatile("" ::: "memory");
    }
    // activation fragments of this wavefront's k-steps: one round trip, straight into registers
    bf16x8 xk[kMaxKW][MT];
#pragma unroll
    for (int ksl = 0; ksl < kMaxKW; ++ksl)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xk[ksl][mt] = buf_load_b(xr, (ksl * MT + mt) * 1024 + lane * 16);
    asm volatile("" ::: "memory");
    if (norm) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < kSsqPer; ++u) s += sv[mt][u];
        s = rows_sum(s);
        if (g == 0) fc.s_part[wave * 64 + mt * 16 + col] = s;
      }
    }
    BD_SUBTS2(1);
    const int mt_e = MT == 1 ? 0 : wave % MT;                // token tile of this wavefront's epilogue elements (4 % MT == 0)
    const int token = mt_e * 16 + col;
    for (int t0 = 0; t0 < n_tiles; t0 += kRound) {
      const int nt = min(kRound, n_tiles - t0);
      const int n_el = nt * MT;                              // (tile, token tile) elements, dealt to the wavefronts
      // operands of the first element's epilogue, fetched while the product runs (rotary factors, old residual values)
      f32x4 pre = f32x4{0.f, 0.f, 0.f, 0.f}, gn = f32x4{1.f, 1.f, 1.f, 1.f};
      f32x4 wsc[3];
      const int r0 = row0 + (t0 + wave / MT) * 16 + 4 * g;   // first row of this lane in element i: r0 + i * (64 / MT)
      if (wave < n_el) {
        if (ph == PH_QKV) {
          if (token < a.M) pre = *reinterpret_cast<const f32x4*>(a.rope + (size_t)token * (D >> 1) + ((r0 % D) >> 1));
        } else if (ph == PH_O) {
          if (token < a.M) pre = *reinterpret_cast<const f32x4*>(a.xv + ((size_t)(2 * fc.layer) * a.Mp + token) * P.H + r0);
          if constexpr (FP8) gn = *reinterpret_cast<const f32x4*>(a.gains + (size_t)(2 * fc.layer + 1) * P.H + r0);
        }
      }
      if constexpr (FP8) {
        const float* ws = a.wscale + (size_t)fc.layer * a.wscale_layer + ws_off;
#pragma unroll
        for (int i = 0; i < 3; ++i)
          wsc[i] = wave + 4 * i < n_el ? *reinterpret_cast<const f32x4*>(ws + r0 + i * (64 / MT)) : f32x4{1.f, 1.f, 1.f, 1.f};
      }
      f32x4 acc[kRound / kT][kT][MT];
#pragma unroll
      for (int c = 0; c < kRound / kT; ++c)
#pragma unroll
        for (int t = 0; t < kT; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[c][t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (KW > 0) {
        const int steps = FP8 ? KW >> 1 : KW;
#pragma unroll
        for (int c = 0; c < kRound / kT; ++c) {
          if (kT * c + 1 < nt) consume_chunk<MT, true, FP8>(rg, sy, xk, steps, acc[c], lane);
          else if (kT * c < nt) consume_chunk<MT, false, FP8>(rg, sy, xk, steps, acc[c], lane);
        }
      }
      if (stream_paced<MT, FP8, LOCAL>() && wave == 0 && t0 + kRound >= n_tiles && ph >= PH_GU) lds_st32(sy.base + SY_PACE * 4, ph == PH_GU ? kPace.gu_end : kPace.down_end);
      BD_SUBTS2(3);
      // The operands fetched for the epilogue are taken here, before its first store: the vector-memory counter is
      // in order, so a wait for them placed behind a write-through store would also wait for that store's
      // acknowledgement (and after a branch that may have stored, the compiler can only wait for everything).
      asm volatile("" ::"v"(pre), "v"(gn));
      if constexpr (FP8) asm volatile("" ::"v"(wsc[0]), "v"(wsc[1]), "v"(wsc[2]));
      // the four consumers hold disjoint K ranges: sum them through LDS in fixed order
      if (t0 > 0) cbar(sy, lane, a.st);                      // (the round before has been read)
#pragma unroll
      for (int c = 0; c < kRound / kT; ++c)
        if (kT * c < nt) {
#pragma unroll
          for (int t = 0; t < kT; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) fc.red[(wave * (kRound * MT) + (c * kT + t) * MT + mt) * 64 + lane] = acc[c][t][mt];
        }
      cbar(sy, lane, a.st);
      BD_SUBTS2(2);
      float rs = 1.f;
      if (norm) {
        const float t = fc.s_part[token] + fc.s_part[64 + token] + fc.s_part[128 + token] + fc.s_part[192 + token];
        rs = rsqrtf(t / (float)P.H + a.rms_eps);
      }
      f32x4 v[3];
      {
        const f32x4* rd = fc.red + wave * 64 + lane;         // (elements that are not there are read and not used)
        f32x4 p[3][kWavesPerWG];
#pragma unroll
        for (int i = 0; i < (kRound * MT + 3) / 4; ++i)
#pragma unroll
          for (int w = 0; w < kWavesPerWG; ++w) p[i][w] = rd[(w * kRound * MT + 4 * i) * 64];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < (kRound * MT + 3) / 4; ++i) {
          v[i] = (p[i][0] + p[i][1] + p[i][2] + p[i][3]) * rs;
          if constexpr (FP8) v[i] *= wsc[i];
        }
      }
      if (ph == PH_GU) {
        // rows (2f, 2f+1) = (gate f, up f): features f, f + 1 of this lane sit side by side
        if (token < a.M) {
          u16* dst = a.act + (size_t)fc.layer * a.act_elems + xp_index(token, r0 >> 1, a.MT);
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            if (wave + 4 * i >= n_el) break;
            const uint32_t h0 = f32_to_bf16_bits(v[i][0] / (1.f + __expf(-v[i][0])) * v[i][1]);
            const uint32_t h1 = f32_to_bf16_bits(v[i][2] / (1.f + __expf(-v[i][2])) * v[i][3]);
            u16* d = i == 0 ? dst : a.act + (size_t)fc.layer * a.act_elems + xp_index(token, (r0 + i * (64 / MT)) >> 1, a.MT);
            if (a.local_gu) *reinterpret_cast<uint32_t*>(d) = h0 | (h1 << 16);   // read only inside this XCD: its L2 is coherent
            else st_wt_u32(d, h0 | (h1 << 16));
          }
        }
      } else if (ph == PH_DOWN) {
        // partial tiles of this K group, in fragment order
        const int kg = blockIdx.x % P.ph[PH_DOWN].ksplit;
        float* dst = a.wsD + (size_t)fc.layer * a.wsD_layer_floats +
                     ((((size_t)kg * (P.H >> 4) + (r0 >> 4)) * MT + mt_e) * 64 + lane) * 4;
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (wave + 4 * i < n_el) st_wt_f32x4(dst + (size_t)i * 4 * 256, v[i]);   // (element el + 4: 4 / MT tiles on)
      } else if (ph == PH_QKV) {
        if (wave < n_el && token < a.M) epilogue_qkv<D>(a, fc, token, r0, v[0], pre);
#pragma unroll 1
        for (int i = 1; wave + 4 * i < n_el; ++i) {          // (plans with more than one element per wavefront)
          v[0] = v[1];
          v[1] = v[2];
          const int r = r0 + i * (64 / MT);
          if (token < a.M)
            epilogue_qkv<D>(a, fc, token, r, v[0], *reinterpret_cast<const f32x4*>(a.rope + (size_t)token * (D >> 1) + ((r % D) >> 1)));
        }
      } else {
        if (wave < n_el) epilogue_residual<FP8>(a, 2 * fc.layer + 1, token, r0, v[0], pre, gn, g);
#pragma unroll 1
        for (int i = 1; wave + 4 * i < n_el; ++i) {
          v[0] = v[1];
          v[1] = v[2];
          const int r = r0 + i * (64 / MT);
          if (token < a.M) pre = *reinterpret_cast<const f32x4*>(a.xv + ((size_t)(2 * fc.layer) * a.Mp + token) * P.H + r);
          if constexpr (FP8) gn = *reinterpret_cast<const f32x4*>(a.gains + (size_t)(2 * fc.layer + 1) * P.H + r);
          epilogue_residual<FP8>(a, 2 * fc.layer + 1, token, r, v[0], pre, gn, g);
        }
      }
      BD_SUBTS2(4);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this wavefront's stores have been acknowledged
  BD_SUBTS2(9);

  if (ph == PH_DOWN && n_tiles > 0) {
    // the last of the ksplit workgroups to finish a tile sums all partials, adds the residual, stores the new
    // residual version and its sum of squares
    const int ksplit = P.ph[PH_DOWN].ksplit;
    const int tiles = P.H >> 4, gt0 = row0 >> 4;
    const int ver = 2 * fc.layer + 2;
    const int n_idx = n_tiles * MT;                           // (tile, row tile of tokens) pairs of this row range
    cbar(sy, lane, a.st);                                    // every consumer's partials are out
    const int t = wave * 64 + lane;
    if (t < n_tiles) {
      int last = 1;
      if (ksplit > 1) {
        const unsigned old = __hip_atomic_fetch_add(a.cntD + (size_t)fc.layer * tiles + gt0 + t, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        last = old == (unsigned)ksplit - 1u;
      }
      fc.s_flags[8 + t] = last;
    }
    cbar(sy, lane, a.st);
    const float* src = a.wsD + (size_t)fc.layer * a.wsD_layer_floats;
    for (int idx0 = wave; idx0 < n_idx; idx0 += 2 * kWavesPerWG) {
      // two pairs per round, every load of the round in flight at once
      f32x4 pv[2][8], xov[2], gnv[2];
      bool on[2];
      int tok[2], rr[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int idx = idx0 + j * kWavesPerWG;
        const int tl = idx / MT, mt = idx % MT;
        on[j] = idx < n_idx && fc.s_flags[8 + min(tl, n_tiles - 1)];
        tok[j] = mt * 16 + col;
        rr[j] = row0 + tl * 16 + 4 * g;
        xov[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        gnv[j] = f32x4{1.f, 1.f, 1.f, 1.f};
        if constexpr (FP8) {
          if (on[j] && ver < 2 * P.L) gnv[j] = *reinterpret_cast<const f32x4*>(a.gains + (size_t)ver * P.H + rr[j]);
        }
        if (on[j]) {
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int kg = min(u, ksplit - 1);
            pv[j][u] = *reinterpret_cast<const f32x4*>(src + ((((size_t)kg * tiles + gt0 + tl) * MT + mt) * 64 + lane) * 4);
          }
          if (tok[j] < a.M) xov[j] = *reinterpret_cast<const f32x4*>(a.xv + ((size_t)(ver - 1) * a.Mp + tok[j]) * P.H + rr[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (!on[j]) continue;
        const int idx = idx0 + j * kWavesPerWG;
        const int tl = idx / MT, mt = idx % MT;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (u < ksplit) v += pv[j][u];
        for (int kg = 8; kg < ksplit; ++kg)
          v += *reinterpret_cast<const f32x4*>(src + ((((size_t)kg * tiles + gt0 + tl) * MT + mt) * 64 + lane) * 4);
        epilogue_residual<FP8>(a, ver, tok[j], rr[j], v, xov[j], gnv[j], g);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    BD_SUBTS2(10);
  }
#undef BD_SUBTS2
}

// ---- attention phase ------------------------------------------------------------------------------------------
// Items (kv head, 16-column tile of (head, token) columns, key chunk).  The four consumers of a workgroup take
// the key blocks of the chunk round-robin, each with its own online softmax, and merge through LDS.  With a
// single chunk (short contexts) the merged result is final and goes straight out; otherwise the partial is
// stored and the workgroup completing the last chunk of a tile merges all chunks in fixed order.
__device__ inline void stream_attn_chunks(int n_keys, int max_chunks, int& n_kb, int& chunk_len, int& n_chunks) {
  n_kb = (n_keys + 31) >> 5;
  int want = n_kb <= 96 ? 1 : (n_kb + 39) / 40;              // short contexts: one chunk (a cross-workgroup merge costs more)
  if (want > max_chunks) want = max_chunks;
  chunk_len = ((n_kb + want - 1) / want + 3) & ~3;
  n_chunks = (n_kb + chunk_len - 1) / chunk_len;
}

template <int D>
struct KvBlock {
  bf16x8 k[2][D / 32];
  bf16x8 v[D / 16];
};

// Block kb of a kv head (the keys of positions 32 kb .. 32 kb + 31) out of the page that holds it.
template <int D>
__device__ inline void kv_load_k(KvBlock<D>& b, const bf16x8* Kh, int page, int lane) {
  constexpr int DS = D / 32;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) b.k[t][ds] = Kh[(((size_t)page * 2 + t) * DS + ds) * 64 + lane];
}
template <int D>
__device__ inline void kv_load_v(KvBlock<D>& b, const bf16x8* Vh, int page, int lane) {
  constexpr int DT = D / 16;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) b.v[dt] = Vh[((size_t)page * DT + dt) * 64 + lane];
}
template <int D>
__device__ inline void kv_load(KvBlock<D>& b, const bf16x8* Kh, const bf16x8* Vh, int kb_logical, int lane, const int* pages) {
  const int kb = page_of_block(pages, __builtin_amdgcn_readfirstlane(kb_logical));
  kv_load_k<D>(b, Kh, kb, lane);
  kv_load_v<D>(b, Vh, kb, lane);
}

// The same through buffer descriptors of the kv head's keys and values, for loops that look ahead: `ok` false requests nothing (an
// offset past the end), but the loads are issued either way, so the compiler knows how many are younger than those it waits
// for.  (Behind a look-ahead that may not have been issued it waits for everything, the look-ahead included: 32 rows, 8192 keys, eight
// blocks per wavefront, one forward 2471 us; in this form 2413 to 2422.)
template <int D>
__device__ inline void kv_load_ahead(KvBlock<D>& b, const rsrc_t& kr, const rsrc_t& vr, int kb_logical, bool ok, int lane, const int* pages) {
  constexpr int DS = D / 32, DT = D / 16;
  const int kb = ok ? page_of_block(pages, __builtin_amdgcn_readfirstlane(kb_logical)) : 0;
  const int off = ok ? kb * (64 * D) + lane * 16 : 0x7FFF0000;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) b.k[t][ds] = buf_load_b(kr, off + (t * DS + ds) * 1024);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) b.v[dt] = buf_load_b(vr, off + dt * 1024);
}

// One block of 32 keys against one tile of 16 query columns.  Scores stay unscaled until the exponent:
// p = 2^(s*c - m) with c = log2(e)/sqrt(d) folded into one fused multiply-add per score.
template <int D, bool MASKED, bool QUAD = false>
__device__ inline void attn_block(const KvBlock<D>& b, const bf16x8 (&qf)[D / 32], f32x4 (&O)[D / 16], float& mrun, float& lrun,
                                  int kb, int n, int M, int mode, int row, int g, float c) {
  constexpr int DS = D / 32, DT = D / 16;
  f32x4 s[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.k[t][ds], qf[ds], s[t], 0, 0, 0);
  }
  float v[8];
  bool vis[8];
  float cmax = kNegBig;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = s[e >> 2][e & 3];
    vis[e] = true;
    if constexpr (MASKED) {
      const int jb = kb * 32 + 8 * g + e - n;
      vis[e] = (jb < 0) || (jb < M && block_key_visible<QUAD>(mode, row, jb));
      if (vis[e]) cmax = fmaxf(cmax, v[e]);
    } else {
      cmax = fmaxf(cmax, v[e]);
    }
  }
  cmax = rows_max(cmax);
  const float mnew = fmaxf(mrun, cmax * c);
  float psum = 0.f;
  bf16x8 p8;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float p = __builtin_amdgcn_exp2f(fmaf(v[e], c, -mnew));
    if constexpr (MASKED) p = vis[e] ? p : 0.f;
    psum += p;
    p8[e] = (__bf16)p;
  }
  psum = rows_sum(psum);
  if (__builtin_amdgcn_ballot_w64(mnew != mrun) != 0ull) {          // some column's maximum moved: rescale
    const float alpha = __builtin_amdgcn_exp2f(mrun - mnew);
    lrun *= alpha;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) O[dt] *= alpha;
    mrun = mnew;
  }
  lrun += psum;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.v[dt], p8, O[dt], 0, 0, 0);
}

template <int D, bool QUAD>
__device__ inline void stream_attention_phase(const MegaArgs& a, FwdCtx& fc, FwdSync& sy, int wave, int lane_in) {
  constexpr int DS = D / 32, DT = D / 16;
  int lane = lane_in;
  asm volatile("" : "+v"(lane));
  const MegaPlan& P = a.P;
  f32x4* sO = reinterpret_cast<f32x4*>(fc.share);                        // [4][DT][64]
  float* sm = reinterpret_cast<float*>(fc.share + kWavesPerWG * DT * 1024);   // [4][16]
  float* sl = sm + kWavesPerWG * 16;                                     // [4][16]
  float* wgt = sl + kWavesPerWG * 16;                                    // [64 chunks][16]
  float* s_inv = wgt + 64 * 16;                                          // [16]

  const int col = lane & 15, g = lane >> 4;
  const int n = fc.n;
  const int G = P.n_q / P.n_kv;
  const int Mp = a.MT * 16;
  const int n_ct = G * a.MT;                                             // column tiles per kv head
  int n_kb, chunk_len, n_chunks;
  const int n_groups = P.n_kv * n_ct;
  stream_attn_chunks(n + a.M, a.attn_max_chunks, n_kb, chunk_len, n_chunks);
  const int n_items = n_groups * n_chunks;
  const size_t kv_block = (size_t)32 * D / 8;
  const u16* Qb = a.Q + (size_t)fc.layer * a.Mp * P.n_q * D;
  float* pO = a.pO + (size_t)fc.layer * a.pO_layer_floats;
  float* pm = a.pm + (size_t)fc.layer * a.pml_layer_floats;
  float* pl = a.pl + (size_t)fc.layer * a.pml_layer_floats;
  u16* out = a.ap + (size_t)fc.layer * a.ap_elems;
  const float c = a.scale_log2e;

#define BD_ATS(k)                                                                                     \
  do {                                                                                                \
    if (a.trace2 != nullptr && fc.layer == 1 && threadIdx.x == 0) a.trace2[(size_t)blockIdx.x * 64 + 48 + (k)] = wall_clock64(); \
  } while (0)
  BD_ATS(0);
  for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int chunk = item % n_chunks;
    const int grp = item / n_chunks;
    const int ct = grp % n_ct, kvh = grp / n_ct;
    const bf16x8* Kh = reinterpret_cast<const bf16x8*>(a.Kc + (size_t)fc.layer * a.kv_layer_elems) + (size_t)kvh * a.max_kb * kv_block;
    const bf16x8* Vh = reinterpret_cast<const bf16x8*>(a.Vc + (size_t)fc.layer * a.kv_layer_elems) + (size_t)kvh * a.max_kb * kv_block;
    const int cidx = ct * 16 + col;
    const int hq = cidx / Mp, row = cidx - hq * Mp;
    bf16x8 qf[DS];
    {
      const u16* qp = Qb + ((size_t)row * P.n_q + kvh * G + hq) * D + 8 * g;
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8*>(qp + ds * 32);
    }
    f32x4 O[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = kNegBig, lrun = 0.f;
    const int kb_end = min(n_kb, (chunk + 1) * chunk_len);
    const int kb0 = chunk * chunk_len + wave;
    // two register buffers, loads pinned one block ahead of their use
    KvBlock<D> b0, b1;
    if (kb0 < kb_end) kv_load<D>(b0, Kh, Vh, kb0, lane, a.kv_pages);
    asm volatile("" ::: "memory");
    for (int kb = kb0; kb < kb_end; kb += 2 * kWavesPerWG) {
      const int kb1 = kb + kWavesPerWG, kb2 = kb + 2 * kWavesPerWG;
      if (kb1 < kb_end) kv_load<D>(b1, Kh, Vh, kb1, lane, a.kv_pages);
      asm volatile("" ::: "memory");
      if (kb * 32 + 31 >= n) attn_block<D, true, QUAD>(b0, qf, O, mrun, lrun, kb, n, a.M, a.mode, row, g, c);
      else attn_block<D, false>(b0, qf, O, mrun, lrun, kb, n, a.M, a.mode, row, g, c);
      if (kb1 < kb_end) {
        if (kb2 < kb_end) kv_load<D>(b0, Kh, Vh, kb2, lane, a.kv_pages);
        asm volatile("" ::: "memory");
        if (kb1 * 32 + 31 >= n) attn_block<D, true, QUAD>(b1, qf, O, mrun, lrun, kb1, n, a.M, a.mode, row, g, c);
        else attn_block<D, false>(b1, qf, O, mrun, lrun, kb1, n, a.M, a.mode, row, g, c);
      }
    }
    BD_ATS(2);
    // merge the four consumers: everyone publishes (max, sum, O), then each folds a share of the d tiles
    if (g == 0) {
      sm[wave * 16 + col] = mrun;
      sl[wave * 16 + col] = lrun;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) sO[(wave * DT + dt) * 64 + lane] = O[dt];
    cbar(sy, lane, a.st);
    BD_ATS(3);
    float mm = sm[col];
#pragma unroll
    for (int w = 1; w < kWavesPerWG; ++w) mm = fmaxf(mm, sm[w * 16 + col]);
    float f[kWavesPerWG];
    float ll = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerWG; ++w) {
      f[w] = exp2f(sm[w * 16 + col] - mm);
      ll += sl[w * 16 + col] * f[w];
    }
    if (n_chunks == 1) {
      const float inv = 1.f / ll;
      for (int dt = wave; dt < DT; dt += kWavesPerWG) {
        f32x4 acc = sO[(0 * DT + dt) * 64 + lane] * f[0];
#pragma unroll
        for (int w = 1; w < kWavesPerWG; ++w) acc += sO[(w * DT + dt) * 64 + lane] * f[w];
        acc *= inv;
        if (row < a.M) {
          const int fo = (kvh * G + hq) * D + dt * 16 + 4 * g;
          const uint32_t lo = (uint32_t)f32_to_bf16_bits(acc[0]) | ((uint32_t)f32_to_bf16_bits(acc[1]) << 16);
          const uint32_t hi = (uint32_t)f32_to_bf16_bits(acc[2]) | ((uint32_t)f32_to_bf16_bits(acc[3]) << 16);
          st_wt_u64(out + xp_index(row, fo, a.MT), (uint64_t)lo | ((uint64_t)hi << 32));
        }
      }
      BD_ATS(4);
      cbar(sy, lane, a.st);                                   // the merge buffers are free again
      continue;
    }
    float* po = pO + (size_t)item * DT * 64 * 4;
    for (int dt = wave; dt < DT; dt += kWavesPerWG) {
      f32x4 acc = sO[(0 * DT + dt) * 64 + lane] * f[0];
#pragma unroll
      for (int w = 1; w < kWavesPerWG; ++w) acc += sO[(w * DT + dt) * 64 + lane] * f[w];
      st_wt_f32x4(po + ((size_t)dt * 64 + lane) * 4, acc);
    }
    if (wave == 0 && g == 0) {
      st_wt_f32(pm + (size_t)item * 16 + col, mm);
      st_wt_f32(pl + (size_t)item * 16 + col, ll);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    cbar(sy, lane, a.st);
    if (wave == 0 && lane == 0) {
      const unsigned old = __hip_atomic_fetch_add(a.cntA + (size_t)fc.layer * n_groups + grp, 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
      fc.s_flags[4] = old == (unsigned)n_chunks - 1u;
    }
    cbar(sy, lane, a.st);
    if (fc.s_flags[4]) {
      // last arriver of this (kv head, column tile): merge all chunks in fixed order
      const size_t item0 = (size_t)grp * n_chunks;
      if (wave == 0) {
        // lane (col, g) looks at chunks g, g+4, ...; at most 64 chunks
        float pmv[16], plv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int ch = g + 4 * u;
          const int chc = min(ch, n_chunks - 1);
          pmv[u] = pm[(item0 + chc) * 16 + col];
          plv[u] = pl[(item0 + chc) * 16 + col];
        }
        float mx = kNegBig;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          if (g + 4 * u >= n_chunks) { pmv[u] = kNegBig; plv[u] = 0.f; }
          mx = fmaxf(mx, pmv[u]);
        }
        mx = rows_max(mx);
        float lp = 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int ch = g + 4 * u;
          const float w = exp2f(pmv[u] - mx);
          lp += plv[u] * w;
          if (ch < n_chunks) wgt[ch * 16 + col] = w;
        }
        lp = rows_sum(lp);
        if (g == 0) s_inv[col] = 1.f / lp;
      }
      cbar(sy, lane, a.st);
      const float* pg = pO + item0 * DT * 64 * 4;
      for (int dt = wave; dt < DT; dt += kWavesPerWG) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int ch0 = 0; ch0 < n_chunks; ch0 += 8) {
          f32x4 pv[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int chc = min(ch0 + u, n_chunks - 1);
            pv[u] = *reinterpret_cast<const f32x4*>(pg + (((size_t)chc * DT + dt) * 64 + lane) * 4);
          }
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (ch0 + u < n_chunks) acc += pv[u] * wgt[(ch0 + u) * 16 + col];
        }
        acc *= s_inv[col];
        if (row < a.M) {
          const int fo = (kvh * G + hq) * D + dt * 16 + 4 * g;
          const uint32_t lo = (uint32_t)f32_to_bf16_bits(acc[0]) | ((uint32_t)f32_to_bf16_bits(acc[1]) << 16);
          const uint32_t hi = (uint32_t)f32_to_bf16_bits(acc[2]) | ((uint32_t)f32_to_bf16_bits(acc[3]) << 16);
          st_wt_u64(out + xp_index(row, fo, a.MT), (uint64_t)lo | ((uint64_t)hi << 32));
        }
      }
    }
    cbar(sy, lane, a.st);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  BD_ATS(5);
#undef BD_ATS
}

// ---- attention phase kept inside each XCD ------------------------------------------------------------------------
// The split over key chunks above pays only for long contexts, because its merge is a chain of far-memory round trips
// (write-through partials, counter, reload by the last arriver).  When workgroup b runs on XCD b mod 8 (the rule the
// gate/up hand-over already relies on) the whole chip can work on a short context instead: the column tiles
// ((head, token) columns, 16 per tile) are dealt out to the XCDs, CT tiles each, all of one kv head; inside an XCD the
// tile's keys are spread over NCH = (workgroups per XCD) / CT workgroups and their four wavefronts (key block kb goes
// to chunk kb mod NCH, wavefront (kb / NCH) mod 4: every wavefront holds one or two blocks of a 1024-token context).
// Partials go to the XCD's L2 with plain stores, the workgroups of the XCD meet at their own barrier, and the merge is
// shared out again: (column tile, 16-dim slice) items over the XCD's wavefronts, each summing the NCH partials of its
// slice in chunk order.  Only the merged bf16 output is written through, for the O projection of all XCDs.
__device__ inline bool stream_xcd_barrier(const MegaArgs& a, FwdSync& sy, unsigned xepoch, int wave, int lane);

template <int D, bool QUAD>
__device__ inline bool stream_attention_local(const MegaArgs& a, FwdCtx& fc, FwdSync& sy, unsigned xepoch, int wave, int lane_in) {
  constexpr int DS = D / 32, DT = D / 16;
  int lane = lane_in;
  asm volatile("" : "+v"(lane));
  const MegaPlan& P = a.P;
  f32x4* sO = reinterpret_cast<f32x4*>(fc.share);                        // [4][DT][64]
  float* sm = reinterpret_cast<float*>(fc.share + kWavesPerWG * DT * 1024);   // [4][16]
  float* sl = sm + kWavesPerWG * 16;                                     // [4][16]

  const int col = lane & 15, g = lane >> 4;
  const int n = fc.n;
  const int G = P.n_q / P.n_kv;
  const int Mp = a.MT * 16;
  const int n_ct = G * a.MT;                                             // column tiles per kv head
  AttnLocalPlan lp;
  attn_local_plan(P.nwg, a.n_xcd, P.n_kv, n_ct, lp);
  const int x = blockIdx.x % a.n_xcd, w = blockIdx.x / a.n_xcd;          // XCD, workgroup inside it
  const int n_kb = (n + a.M + 31) >> 5;
  const size_t kv_block = (size_t)32 * D / 8;
  const u16* Qb = a.Q + (size_t)fc.layer * a.Mp * P.n_q * D;
  float* pO = a.pO + (size_t)fc.layer * a.pO_layer_floats;
  float* pm = a.pm + (size_t)fc.layer * a.pml_layer_floats;
  float* pl = a.pl + (size_t)fc.layer * a.pml_layer_floats;
  u16* out = a.ap + (size_t)fc.layer * a.ap_elems;
  const float c = a.scale_log2e;

#define BD_ATS(k)                                                                                     \
  do {                                                                                                \
    if (a.trace2 != nullptr && fc.layer == 1 && threadIdx.x == 0) a.trace2[(size_t)blockIdx.x * 64 + 48 + (k)] = wall_clock64(); \
  } while (0)
  BD_ATS(0);
  {
    const int ctl = w % lp.CT, chunk = w / lp.CT;
    const int ct = x * lp.CT + ctl;                                      // column tile of this workgroup
    const int kvh = ct / n_ct, ctk = ct - kvh * n_ct;
    const bf16x8* Kh = reinterpret_cast<const bf16x8*>(a.Kc + (size_t)fc.layer * a.kv_layer_elems) + (size_t)kvh * a.max_kb * kv_block;
    const bf16x8* Vh = reinterpret_cast<const bf16x8*>(a.Vc + (size_t)fc.layer * a.kv_layer_elems) + (size_t)kvh * a.max_kb * kv_block;
    const int cidx = ctk * 16 + col;
    const int hq = cidx / Mp, row = cidx - hq * Mp;
    bf16x8 qf[DS];
    {
      const u16* qp = Qb + ((size_t)row * P.n_q + kvh * G + hq) * D + 8 * g;
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8*>(qp + ds * 32);
    }
    f32x4 O[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = kNegBig, lrun = 0.f;
    const int stride = kWavesPerWG * lp.NCH;
    const int kb0 = chunk + lp.NCH * wave;
    const rsrc_t kr = make_rsrc(Kh, (unsigned)(a.max_kb * 64 * D)), vr = make_rsrc(Vh, (unsigned)(a.max_kb * 64 * D));
    KvBlock<D> b0, b1;
    kv_load_ahead<D>(b0, kr, vr, kb0, kb0 < n_kb, lane, a.kv_pages);
    asm volatile("" ::: "memory");
    for (int kb = kb0; kb < n_kb; kb += 2 * stride) {
      const int kb1 = kb + stride, kb2 = kb + 2 * stride;
      kv_load_ahead<D>(b1, kr, vr, kb1, kb1 < n_kb, lane, a.kv_pages);
      asm volatile("" ::: "memory");
      if (kb * 32 + 31 >= n) attn_block<D, true, QUAD>(b0, qf, O, mrun, lrun, kb, n, a.M, a.mode, row, g, c);
      else attn_block<D, false>(b0, qf, O, mrun, lrun, kb, n, a.M, a.mode, row, g, c);
      if (kb1 < n_kb) {
        kv_load_ahead<D>(b0, kr, vr, kb2, kb2 < n_kb, lane, a.kv_pages);
        asm volatile("" ::: "memory");
        if (kb1 * 32 + 31 >= n) attn_block<D, true, QUAD>(b1, qf, O, mrun, lrun, kb1, n, a.M, a.mode, row, g, c);
        else attn_block<D, false>(b1, qf, O, mrun, lrun, kb1, n, a.M, a.mode, row, g, c);
      }
    }
    BD_ATS(2);
    // merge the four consumers through LDS, each folding a share of the d tiles; the result is this workgroup's partial
    if (g == 0) {
      sm[wave * 16 + col] = mrun;
      sl[wave * 16 + col] = lrun;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) sO[(wave * DT + dt) * 64 + lane] = O[dt];
    cbar(sy, lane, a.st);
    float mm = sm[col];
#pragma unroll
    for (int wv = 1; wv < kWavesPerWG; ++wv) mm = fmaxf(mm, sm[wv * 16 + col]);
    float f[kWavesPerWG];
    float ll = 0.f;
#pragma unroll
    for (int wv = 0; wv < kWavesPerWG; ++wv) {
      f[wv] = exp2f(sm[wv * 16 + col] - mm);
      ll += sl[wv * 16 + col] * f[wv];
    }
    float* po = pO + (size_t)blockIdx.x * DT * 64 * 4;
    for (int dt = wave; dt < DT; dt += kWavesPerWG) {
      f32x4 acc = sO[(0 * DT + dt) * 64 + lane] * f[0];
#pragma unroll
      for (int wv = 1; wv < kWavesPerWG; ++wv) acc += sO[(wv * DT + dt) * 64 + lane] * f[wv];
      *reinterpret_cast<f32x4*>(po + ((size_t)dt * 64 + lane) * 4) = acc;   // read only inside this XCD: its L2 is coherent
    }
    if (wave == 0 && g == 0) {
      pm[(size_t)blockIdx.x * 16 + col] = mm;
      pl[(size_t)blockIdx.x * 16 + col] = ll;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    BD_ATS(3);
  }
  if (!stream_xcd_barrier(a, sy, xepoch, wave, lane)) return false;
  BD_ATS(4);
  // merge: item (column tile ctl, d tile dt) -> workgroup item mod WX, wavefront item / WX
  for (int item = w + lp.WX * wave; item < lp.CT * DT; item += lp.WX * kWavesPerWG) {
    const int ctl = item / DT, dt = item - ctl * DT;
    const int ct = x * lp.CT + ctl;
    const int kvh = ct / n_ct, ctk = ct - kvh * n_ct;
    const int cidx = ctk * 16 + col;
    const int hq = cidx / Mp, row = cidx - hq * Mp;
    // partial of chunk ch of this tile: the workgroup with w = ch * CT + ctl of this XCD.  Eight chunks per batch, and
    // two batches requested before the first is used (up to 16 chunks, all that a forward of at most 16 rows has, cost
    // one round trip to the L2); a running maximum carries from batch to batch, chunks in order.  What bounds the merge
    // is that latency: with a loop over the maxima ahead of the loads (one round trip per chunk) the phase took 12.0 us
    // per layer at 1 row and 10.5 at 32 rows (1024 keys), a forward 2270 and 2512 us; in this form 2116 and 2422 us.
    float mx = kNegBig, lsum = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Batch { f32x4 o[8]; float m[8], l[8]; };
    auto fetch = [&](Batch& b, int ch0) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const size_t it = (size_t)((min(ch0 + u, lp.NCH - 1) * lp.CT + ctl) * a.n_xcd + x);
        b.m[u] = pm[it * 16 + col];
        b.l[u] = pl[it * 16 + col];
        b.o[u] = *reinterpret_cast<const f32x4*>(pO + (it * DT + dt) * 64 * 4 + (size_t)lane * 4);
      }
    };
    auto fold = [&](const Batch& b, int ch0) {
      float mn = mx;
#pragma unroll
      for (int u = 0; u < 8; ++u) mn = fmaxf(mn, b.m[u]);                // (a repeated last chunk does not move the maximum)
      const float f = exp2f(mx - mn);
      acc *= f;
      lsum *= f;
      mx = mn;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float wq = ch0 + u < lp.NCH ? exp2f(b.m[u] - mn) : 0.f;
        acc += b.o[u] * wq;
        lsum += b.l[u] * wq;
      }
    };
    for (int ch0 = 0; ch0 < lp.NCH; ch0 += 16) {
      Batch b0, b1;
      fetch(b0, ch0);
      if (ch0 + 8 < lp.NCH) fetch(b1, ch0 + 8);
      fold(b0, ch0);
      if (ch0 + 8 < lp.NCH) fold(b1, ch0 + 8);
    }
    acc *= 1.f / lsum;
    if (row < a.M) {
      const int fo = (kvh * G + hq) * D + dt * 16 + 4 * g;
      const uint32_t lo = (uint32_t)f32_to_bf16_bits(acc[0]) | ((uint32_t)f32_to_bf16_bits(acc[1]) << 16);
      const uint32_t hi = (uint32_t)f32_to_bf16_bits(acc[2]) | ((uint32_t)f32_to_bf16_bits(acc[3]) << 16);
      st_wt_u64(out + xp_index(row, fo, a.MT), (uint64_t)lo | ((uint64_t)hi << 32));
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  BD_ATS(5);
#undef BD_ATS
  return true;
}

// ---- grid barrier of the consumer wavefronts ---------------------------------------------------------------------
// Every consumer has waited for its own stores (each phase ends with that wait).  Consumer 0 collects the four
// arrivals, takes part in the chip-wide barrier (key split: two-level counters of mega.h) and hands the new epoch to the
// others through LDS.
// LOCAL: the workgroups of an XCD meet at a counter in its L2, and the last one there writes the epoch into its word of every
// XCD's line (a.xbar: lines 8.. hold the counters, lines 16.. the words), which the workgroups of that XCD poll: one far
// round trip behind the last arrival instead of three (two levels of far counters, release).  All workgroups arriving at once: 1.59
// us against 1.65, with a store before and a load behind it 3.05 against 3.18, and more beside the stream, where every far round trip
// is longer.  One forward, 3B shape: 4 rows 1884 -> 1827 us, 32 rows 2009 -> 1962 (1024 keys); e4m3 16 rows 1586 -> 1511, 32 rows
// 1978 -> 1934 (333 keys).
template <bool LOCAL>
__device__ inline bool stream_grid_barrier(const MegaArgs& a, FwdSync& sy, unsigned epoch, int wave, int lane_in) {
  int lane = lane_in;
  asm volatile("" : "+v"(lane));                            // (or the addresses below are kept in registers across the phases)
  const int nwg = a.P.nwg;
  sy.arrive_target += kWavesPerWG;
  if (lane == 0) lds_inc(sy.base + SY_ARRIVE * 4);
  if (wave == 0) {
    bool ok = lds_wait_ge(sy, sy.base + SY_ARRIVE * 4, sy.arrive_target, a.st);
    if constexpr (LOCAL) {
      if (ok) {
        const int nx = a.n_xcd, x = blockIdx.x % nx;
        unsigned old = 0u;
        if (lane == 0) old = __hip_atomic_fetch_add(a.xbar + 32 * (8 + x), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        old = (unsigned)__builtin_amdgcn_readfirstlane((int)old);
        if (old == epoch * (unsigned)(nwg / nx) - 1u && lane < nx)
          __hip_atomic_store(a.xbar + 32 * (16 + lane) + x, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned* mine = a.xbar + 32 * (16 + x) + lane % nx;
        int spins = 0;
        while (__builtin_amdgcn_ballot_w64(!counter_reached(__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), epoch)) != 0ull) {
          if (++spins > kSpinLimit) { ok = false; break; }
          __builtin_amdgcn_s_sleep(1);
        }
        if (ok) lds_st32(sy.base + SY_EPOCH * 4, epoch);
        else lds_st32(sy.base + SY_DEAD * 4, kDeadChip);
      }
    } else if (ok && lane == 0) {
      const int ng = (nwg + kBarGroup - 1) / kBarGroup;
      const int g = blockIdx.x / kBarGroup;
      const int gsize = min(kBarGroup, nwg - g * kBarGroup);
      unsigned* gcnt = a.bar + 32 * (1 + g);
      unsigned* rel = a.bar + 32 * (1 + ng);
      const unsigned old = __hip_atomic_fetch_add(gcnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old == epoch * (unsigned)gsize - 1u) {
        const unsigned o2 = __hip_atomic_fetch_add(a.bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (o2 == epoch * (unsigned)ng - 1u)
          for (int r = 0; r < ng; ++r) __hip_atomic_store(rel + 32 * r, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      const unsigned* mine = rel + 32 * g;
      int spins = 0;
      while (!counter_reached(__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), epoch)) {
        if (++spins > kSpinLimit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      if (ok) lds_st32(sy.base + SY_EPOCH * 4, epoch);
      else lds_st32(sy.base + SY_DEAD * 4, kDeadChip);
    }
  }
  const bool ok = lds_wait_ge(sy, sy.base + SY_EPOCH * 4, epoch, a.st);
  asm volatile("" ::: "memory");
  return ok;
}

// ---- barrier of the workgroups of one XCD ------------------------------------------------------------------------
// Workgroup b runs on XCD b mod 8 (checked when the kernel starts), and the CUs of one XCD share one L2.  Between
// workgroups of one XCD a hand-over therefore needs no write-through: plain stores are complete (s_waitcnt) once that
// L2 holds them, and every later load from a CU of the same XCD that misses its L1 reads them there.  The arrival
// counter of XCD x is touched by the workgroups of XCD x only, through read-modify-write atomics, which never execute
// in an L1.
__device__ inline unsigned xcc_id() {
  unsigned x;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
  return x & 15u;
}
__device__ inline unsigned l2_atomic_peek(unsigned* p) {
  unsigned v;
  const unsigned zero = 0u;
  asm volatile("global_atomic_or %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p), "v"(zero) : "memory");
  return v;
}
__device__ inline bool stream_xcd_barrier(const MegaArgs& a, FwdSync& sy, unsigned xepoch, int wave, int lane) {
  sy.arrive_target += kWavesPerWG;
  if (lane == 0) lds_inc(sy.base + SY_ARRIVE * 4);
  if (wave == 0) {
    bool ok = lds_wait_ge(sy, sy.base + SY_ARRIVE * 4, sy.arrive_target, a.st);
    if (ok && lane == 0) {
      const int nx = a.n_xcd;
      unsigned* cnt = a.xbar + 32 * (blockIdx.x % nx);
      const unsigned target = xepoch * (unsigned)(a.P.nwg / nx);
      __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      int spins = 0;
      while (!counter_reached(l2_atomic_peek(cnt), target)) {
        if (++spins > kSpinLimit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(1);
      }
      if (ok) lds_st32(sy.base + SY_XEPOCH * 4, xepoch);
      else {
        lds_st32(sy.base + SY_DEAD * 4, kDeadReported);
        __hip_atomic_store(&a.st->error[DE_XCD_BARRIER], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  const bool ok = lds_wait_ge(sy, sy.base + SY_XEPOCH * 4, xepoch, a.st);
  asm volatile("" ::: "memory");
  return ok;
}

// ---- the kernel ------------------------------------------------------------------------------------------------
template <int MT> constexpr int stream_lds_bytes() { return kWavesPerWG * kRingBytes + kShareBytes; }

// LOCAL: the attention that stays inside each XCD, else the chip-wide key split.  One of them per instantiation: with both
// compiled in the kernel was 70 KB with 376 B of scratch per lane, with one 52 KB and 80 B (3B shape, 1024 keys, 32 rows: a
// forward 2151 us, with one 2139; up to 16 rows 1970 and 1962; e4m3, 32 rows, 333 keys 2031 and 2064, for the better with the
// pace per phase above).
template <int MT, int D, bool FP8, bool QUAD, bool LOCAL>
__global__ __launch_bounds__(kFwdThreads, 1) void stream_fwd_kernel(MegaArgs a) {
  constexpr int kRound = round_tiles<MT>();
  static_assert(kWavesPerWG * kRound * MT * 1024 <= kShareBytes, "K-reduction buffers exceed the shared region");
  static_assert(kRound * MT <= 3 * kWavesPerWG && kWavesPerWG % MT == 0, "at most three epilogue elements per consumer and round");
  static_assert(kWavesPerWG * (D / 16) * 1024 + (8 * 16 + 64 * 16 + 16) * 4 <= kShareBytes, "attention merge buffers exceed the shared region");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ unsigned s_sync[SY_WORDS];
  __shared__ int s_flags[kFlagWords];
  __shared__ float s_part[kWavesPerWG * 64];
  __shared__ int4 s_plan[PH_LM * kWavesPerWG];
  const MegaPlan& P = a.P;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (threadIdx.x < SY_WORDS) s_sync[threadIdx.x] = sync_word_at_start(threadIdx.x, stream_pace<MT, FP8, LOCAL>().qkv, a.bar_epoch, a.xbar_epoch);
  if (threadIdx.x < PH_LM * kWavesPerWG)
    s_plan[threadIdx.x] = a.wtab[blockIdx.x * kWavesPerWG + threadIdx.x % kWavesPerWG].ph[threadIdx.x / kWavesPerWG];
  if (threadIdx.x == 0) {
    int go = usable(a.st);
    if (go && a.skippable && a.st->skip) {
      const unsigned n_chip = (a.local_gu ? 4u : 5u) * (unsigned)P.L, n_xcd = ((a.local_gu ? 1u : 0u) + (LOCAL ? 1u : 0u)) * (unsigned)P.L;
      if constexpr (LOCAL) {                               // (the words of the lines stay behind; the next real barrier overwrites them)
        __hip_atomic_fetch_add(a.xbar + 32 * (8 + blockIdx.x % a.n_xcd), n_chip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(a.xbar + 32 * (blockIdx.x % a.n_xcd), n_xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        skip_barriers(a.bar, a.xbar, n_chip, n_xcd);
      }
      go = 0;
    }
    if (go && (a.local_gu || LOCAL) && xcc_id() != blockIdx.x % 8u) {   // the XCD-local hand-overs would be unsafe
      __hip_atomic_store(&a.st->error[DE_OTHER], DE_OTHER_XCD, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      go = 0;
    }
    s_flags[0] = go;
  }
  __syncthreads();                                       // the only workgroup barrier: all eight wavefronts are still here
  if (!s_flags[0]) return;
  const unsigned sync_base = lds_addr(s_sync);

  if (wave >= kWavesPerWG) {
    const int cw = wave - kWavesPerWG;
    producer_loop_stash<kStash, MT, FP8, LOCAL>(a, cw, lds + cw * kRingBytes, sync_base, lane);
    return;
  }

  FwdSync sy;
  sy.base = sync_base; sy.cbar_target = 0u; sy.arrive_target = 0u; sy.dead = false;
  Ring rg;
  rg.base = lds + wave * kRingBytes;
  rg.landed_addr = sync_base + (SY_LANDED + wave) * 4;
  rg.consumed_addr = sync_base + (SY_CONSUMED + wave) * 4;
  rg.have = 0u; rg.taken = 0u; rg.slot = 0;
  FwdCtx fc;
  fc.share = lds + kWavesPerWG * kRingBytes;
  fc.n = a.st->n;
  for (int i = 0; i < 3; ++i) fc.pg[i] = page_of_block(a.kv_pages, min((fc.n >> 5) + i, a.max_kb - 1));
  fc.red = reinterpret_cast<f32x4*>(fc.share);
  fc.s_flags = s_flags;
  fc.s_part = s_part;
  fc.s_plan = s_plan;
  unsigned epoch = a.bar_epoch, xepoch = a.xbar_epoch;

  int tsi = 0;
#define BD_TS2()                                                                                                  \
  do {                                                                                                            \
    if (a.trace != nullptr && threadIdx.x == 0) a.trace[(size_t)blockIdx.x * (10 * P.L + 4) + tsi] = wall_clock64(); \
    ++tsi;                                                                                                        \
  } while (0)
  BD_TS2();
  bool alive = true;
  for (int l = 0; l < P.L && alive; ++l) {
    fc.layer = l;
    // the five phases of a layer (QKV, attention, O, gate/up, down), each ended by a barrier: `step` stays a runtime value
    // so that the phases share one copy of the code
#pragma unroll 1
    for (int step = 0; step < 5; ++step) {
      asm volatile("" : "+s"(step));
      if (step == 1) {
        if (stream_paced<MT, FP8, LOCAL>() && wave == 0) lds_st32(sync_base + SY_PACE * 4, stream_pace<MT, FP8, LOCAL>().attn);
        if constexpr (LOCAL) {
          alive = stream_attention_local<D, QUAD>(a, fc, sy, ++xepoch, wave, lane);
          if (!alive) break;
        } else {
          stream_attention_phase<D, QUAD>(a, fc, sy, wave, lane);
        }
      } else {
        stream_gemm_phase<MT, D, FP8, LOCAL>(a, fc, rg, sy, step == 0 ? (int)PH_QKV : step - 1, wave, lane);
      }
      BD_TS2();
      if (step == 3 && a.local_gu) alive = stream_xcd_barrier(a, sy, ++xepoch, wave, lane);
      else alive = stream_grid_barrier<LOCAL>(a, sy, ++epoch, wave, lane);
      BD_TS2();
      if (!alive) break;
    }
  }
  if (sy.dead && lane == 0) {
    const unsigned why = lds_ld32(sync_base + SY_DEAD * 4);
    if (why > (unsigned)kDeadReported) __hip_atomic_store(a.st->error + (why & 3u), (int)DE_RING, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // (SY_DEAD is set by whoever gave up first, so the producers leave too)
#undef BD_TS2
}

}  // namespace bd
