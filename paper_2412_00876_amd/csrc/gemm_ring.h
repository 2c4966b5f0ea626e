// 256 x (32*JT) x d tile product on the matrix cores for the large bfloat16 products of the path (predictor scoring
// over all vision tokens, Q/K/V projection of the kept rows, the linear layers): one block of 4 waves per compute unit,
//   acc[i][j] (16 x 16) += A[128*(w/2) + 16*i + 0..15, :] . B[16*JT*(w%2) + 16*j + 0..15, :]^T ,   i < 8, j < JT,
// for wave w (2 x 2 waves: 128 rows of the 256-row A tile against half of the 32*JT rows of the B tile), with
// v_mfma_f32_16x16x32_bf16.  Both operands are contiguous along d and are streamed in 64-element stages (one whole
// 128-byte memory line per row).
//
// What shapes the loop (each point is a measurement on MI355X, not a guess):
//  * The chip is POWER-bound here, not issue-bound: with normally distributed operands in registers and nothing else
//    running, v_mfma_f32_32x32x16_bf16 holds 1.74 GHz (1767 TFLOP/s) and v_mfma_f32_16x16x32_bf16 2.03 GHz (2041
//    TFLOP/s; both 2450 with zeros): the small shape moves half the accumulator bytes per product.  For the same
//    reason the wave tile is square, 128 x 128: 16 KiB of LDS fragments per 64 products instead of the 20 KiB of
//    64 x 256.  Measured per 256 x 256 block of the Q/K/V projection (64 stages): 102 us at 1.56 GHz with 32x32x16 on
//    64 x 256 wave tiles, 95 us at 1.64 GHz with this form.
//  * A compute unit pulls its operands from L2 at 40-45 bytes per clock at best, so the tile must be large: 256 x 256
//    needs 32 bytes per clock at the full matrix rate, 128 x 128 twice that.  The accumulators of the wave tile
//    fill the 256 accumulation registers; one wave per SIMD.
//  * Tiles go from global memory straight into LDS (global_load_lds_dwordx4, no staging registers).  A stage is 64 KiB,
//    LDS holds 160 KiB, and a tile requested one stage ahead does not arrive in time (latency plus transfer exceed a
//    stage's arithmetic), so the LDS is a ring of FIVE 32 KiB half-stage slots (B, A, B, A, ...): while stage k is
//    multiplied, A of stage k+1 and B of stages k+1 and k+2 are in flight or landed -- every tile is requested
//    a whole stage before the barrier that needs it.
//  * A wave issues in order and there is one wave per SIMD: whatever stands between two products idles the matrix
//    pipe.  Fragment reads and tile loads are dealt out between the products (a burst of loads stalls the wave: the
//    memory pipeline accepts about one 1 KiB load per 25 clocks per compute unit), scheduling barriers keep the
//    compiler from regrouping them, and the scalar arithmetic of the next stage's addresses hides behind products too.
//  * The stage barrier sits before the LAST k-step of a stage: by then the fragments of that k-step are in
//    registers, so the stage's slots are free, and the first fragments of the next stage are read behind the
//    products of the last k-step instead of after a barrier with nothing to hide them.
//  * The products are written as instructions with their accumulators pinned to accumulation registers: with the
//    builtin the compiler kept some of the 64 four-register accumulators in vector registers and moved them back and
//    forth in the loop (400 moves per stage, 3.3 times slower).
// LDS layout of a slot: row r at r*128 bytes, 16-byte chunk c of the row at position c ^ ((r/2) % 8): the 16 lanes
// that the LDS serves together hit 16 different bank groups both when a tile load deposits 8 rows x 8 chunks and
// when a fragment read takes one chunk of 16 rows.
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"

namespace dllava {

typedef float ring_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t ring_u32x4 __attribute__((ext_vector_type(4)));

#define DLLAVA_LDS __attribute__((address_space(3)))
#define DLLAVA_GLB __attribute__((address_space(1)))
#define DLLAVA_INLINE __attribute__((always_inline))

constexpr int kRingThreads = 256;
constexpr int kRingBK = 64;                       // elements of d per stage
constexpr int kRingRowBytes = 128;                // bytes per row per stage
constexpr int kRingSlotBytes = 256 * kRingRowBytes;
constexpr int kRingSlots = 5;
constexpr int kRingLdsBytes = kRingSlots * kRingSlotBytes;  // 160 KiB: all of a compute unit's LDS

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {  // f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

template <int OFF>
__device__ __forceinline__ ring_u32x4 ring_lds_read16(uint32_t addr) {
  ring_u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
__device__ __forceinline__ void ring_mfma(ring_f32x4& c, const ring_u32x4& a, const ring_u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void ring_tie_acc(ring_f32x4& c) { asm volatile("" : "+a"(c)); }

// Byte offset, from the first row of a tile, of the 16 bytes that this lane fetches with tile load j of wave w:
// the load covers rows 8*(w + 4j) + lane/8, the lane's position lane%8 holds chunk (lane%8) ^ ((row/2)%8).
// `row_of(r)` maps tile row r to the row of the matrix (clamping and gathering are the caller's).
__device__ __forceinline__ int ring_load_row(int w, int j, int lane) { return 8 * (w + 4 * j) + (lane >> 3); }
__device__ __forceinline__ uint32_t ring_load_chunk_bytes(int row, int lane) {
  return 16u * static_cast<uint32_t>((lane & 7) ^ ((row >> 1) & 7));
}

// The fragment registers pass through the waiting statement, so nothing that uses them can be scheduled above it.
template <int N>
__device__ __forceinline__ void ring_tie(ring_u32x4 (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
}

// Tile order.  Tiles (A tile at, B tile bt) are numbered in groups of kRingGroup B tiles, inside a group A tile by A
// tile, and XCD x (blocks x, x + 8, ...) takes the x-th eighth of that order: the 32 tiles that an XCD works on at a time
// then cover about 6 A tiles x 5 B tiles, the square patch that pulls the fewest bytes through its L2, and the XCDs
// are loaded alike whatever the numbers of tiles.  False: this block has no tile.
constexpr int kRingXcds = 8;
constexpr int kRingGroup = 5;
__device__ __forceinline__ bool ring_tile(int n_at, int n_bt, int per_xcd, int& at, int& bt) {
  const int xcd = blockIdx.x % kRingXcds, local = blockIdx.x / kRingXcds;
  const int64_t idx = static_cast<int64_t>(xcd) * per_xcd + local;
  if (local >= per_xcd || idx >= static_cast<int64_t>(n_at) * n_bt) return false;
  const int per_group = kRingGroup * n_at;
  const int group = static_cast<int>(idx / per_group), in_group = static_cast<int>(idx % per_group);
  const int left = n_bt - group * kRingGroup, here = left < kRingGroup ? left : kRingGroup;
  at = in_group / here;
  bt = group * kRingGroup + in_group % here;
  return true;
}

// The tiles of the products below: 32*fi rows of A x 32*jt rows of B.  Nanoseconds per stage when every compute unit works and
// when few do -- the clock gives way to the power --, beside the stages (prologue and epilogue), and what the tile loads of a
// stage alone take (measured on linear layers of d = 512 .. 11008).  Blocks that share a compute unit: one; three of the shallow
// small tiles (times: of a whole round of them); two of the tiles that stand with GELU (see ring_pick).  Of the small tile with the
// deep ring, which has half of the LDS, two blocks may stand in a compute unit as well; it is priced as if there were one.
struct RingTile {
  int id;  // what the launch overrides take
  int fi, jt;
  int64_t busy, alone, ends, load;
  int per_cu;
};
constexpr int kRingGeluPair = 12;
constexpr RingTile kRingTiles[] = {{8, 8, 8, 1310, 990, 10200, 800, 1}, {7, 8, 7, 1120, 855, 9300, 750, 1},  {6, 8, 6, 1030, 760, 8400, 700, 1},
                                   {5, 8, 5, 870, 660, 7300, 650, 1},   {4, 8, 4, 750, 600, 6300, 600, 1},   {9, 4, 6, 540, 430, 7500, 430, 1},
                                   {3, 4, 4, 460, 370, 6200, 370, 1},   {10, 4, 2, 300, 270, 4700, 270, 1},  {2, 2, 4, 300, 260, 4500, 260, 1},
                                   {1, 2, 2, 210, 190, 3800, 200, 1},   {11, 2, 2, 700, 210, 3400, 200, 3},  {kRingGeluPair, 4, 4, 800, 460, 5500, 740, 2}};

// The tile that takes least; tiles_of(t): how many of it the launch has, 0 if it cannot use it.  Null if none can be used.
// A stage touches one 128-byte line of every row of its tile: once those rows span more than about 2.5 MiB (11008
// columns: 22 KiB apart) its loads slow down, by about 65 ns for every further MiB -- 4096 x 500 results: 0.98 us a stage
// of 256 x 128 at 11008 columns against 0.60 at 4096, 0.25 against 0.20 of 64 x 64.
// gelu: the epilogue takes the GELU of 4 fi jt results per lane, 32 ns each (vector arithmetic, nothing beside it).  Only then do
// two blocks per compute unit pay, one's products beside the other's GELU: they are paced by the LDS, which two tiles of 128 x 128
// read and write 1.4 times as much per product as one of 256 x 256 (11520 rows, 512 wide: 2048 features with GELU 40.5 us against
// 45.8, 1536 without, over cards, 27.7 to 31.5 against 28.0 to 29.7).  Two blocks of a compute unit that start together stay in
// step, so the first of their rounds of 512 takes 5 us more (and a launch of one round never pays); what is left for a last round
// of at most 256 runs alone, which takes half of the ends.  (4096 features, 544 / 1056 / 1568 tiles: 512 wide 22 / 34 / 45 us, priced
// 23 / 35 / 47; 11008 wide 222 / 360 / 501, priced 253 / 419 / 584, where 256 x 160 takes 149 / 293 and 256 x 224 392, priced
// 206 / 388 / 446.)
template <typename F>
inline const RingTile* ring_pick(int64_t d, int forced, F&& tiles_of, bool gelu = false) {
  const int64_t nk = d / kRingBK;
  const RingTile* best = nullptr;
  int64_t best_cost = 0;
  for (const RingTile& t : kRingTiles) {
    const int64_t tiles = tiles_of(t);
    if (tiles <= 0) continue;
    if (t.id == forced) return &t;
    const int64_t span = 32 * (t.fi + t.jt) * d * 2 - (5 << 19), slow = t.load + (span > 0 ? span / (1 << 10) * 65 / (1 << 10) : 0);
    const int64_t busy = t.busy > slow ? t.busy : slow, alone = t.alone > slow ? t.alone : slow;
    const int64_t at_once = 32 * t.per_cu, per_xcd = ceil_div(tiles, kRingXcds), full = per_xcd / at_once, rest = per_xcd % at_once;
    int64_t cost;
    if (t.id == kRingGeluPair) {
      if (!gelu || tiles <= 512) continue;  // within one round the blocks of a compute unit stay in step: nothing of one stands beside the other
      const int64_t single = t.alone > slow / 2 ? t.alone : slow / 2;
      cost = 5000 + full * (nk * busy + t.ends);
      if (rest) cost += rest > 32 ? nk * busy + t.ends : nk * single + t.ends / 2;
    } else {
      const int64_t ends = t.ends + (gelu ? 4 * 32 * t.fi * t.jt : 0);
      cost = full * (nk * busy + ends);
      if (rest) cost += nk * (alone + (busy - alone) * rest / at_once) + ends;
    }
    if (!best || cost < best_cost) best = &t, best_cost = cost;
  }
  return best;
}

// Main loop, A tile of 32*FI rows, a ring of five half-stage slots of 32*FI rows (FI = 8: all of the LDS, FI = 4: half of it, for two
// blocks per compute unit).  Abase / Bbase: wave-uniform byte pointers to element 0 of the tiles' first rows; ga[j] / gb[j]: this
// lane's byte offsets (ring_load_row / ring_load_chunk_bytes) for its tile loads; nk = d / 64 >= 1;
// w = wave index 0..3 (wave-uniform).  acc: register r of acc[i][j] in a lane is
//   A row 16*FI*(w/2) + 16*i + 4*(lane/16) + r  .  B row 16*JT*(w%2) + 16*j + lane%16.
// Every row touched must be readable for all d (clamp rows past the end of a matrix to its last row).
// On return all LDS traffic of the loop has completed; the caller must still place a block barrier before it
// reuses the ring memory for something else.
// BOff: uint32_t, or int64_t when the rows of B may lie more than 4 GiB apart (gathered rows).
template <int FI, int JT, typename AOff, typename BOff>
__device__ __forceinline__ void gemm_ring_halves(const char* Abase, const AOff (&ga)[FI], const char* Bbase,
                                                 const BOff (&gb)[JT], int nk, DLLAVA_LDS char* smem, int w,
                                                 ring_f32x4 (&acc)[FI][JT]) {
  static_assert(JT >= 4 && JT <= FI, "a slot holds the rows of either tile");
  constexpr int kMF = FI * JT;  // products per k-step of 32
  constexpr int kNR = FI + JT;  // fragment reads per k-step
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t s0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  // fragment of k-step ks: chunk 4*ks + lane/16 of row lane%16 (+ multiples of 16): ks enters as an exclusive-or with 64*ks
  const uint32_t fo = (lane & 15) * kRingRowBytes + (((lane >> 4) ^ ((lane & 15) >> 1)) * 16);
  const uint32_t a_at = s0 + (w >> 1) * (16 * FI) * kRingRowBytes + fo, b_at = s0 + (w & 1) * (16 * JT) * kRingRowBytes + fo;

  ring_u32x4 ua[FI], ub[JT], va[FI], vb[JT];  // two fragment sets: one is multiplied while the other is read

  // stages past the end re-read the last one (in bounds, unused)
  auto koff = [&](int kt) DLLAVA_INLINE { return static_cast<int64_t>(kt < nk ? kt : nk - 1) * (kRingBK * 2); };
  auto dma = [&](const char* src, uint32_t slot, int j) DLLAVA_INLINE {
    __builtin_amdgcn_global_load_lds((const DLLAVA_GLB void*)src,
                                     (DLLAVA_LDS void*)(smem + slot + (w + 4 * j) * 1024), 16, 0, 0);
  };
  auto read1 = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[JT], uint32_t ab, uint32_t bb, auto I) DLLAVA_INLINE {
    constexpr int i = decltype(I)::value;
    if constexpr (i < FI)
      fa[i] = ring_lds_read16<i * 16 * kRingRowBytes>(ab);
    else
      fb[i - FI] = ring_lds_read16<(i - FI) * 16 * kRingRowBytes>(bb);
  };
  auto wait = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[JT]) DLLAVA_INLINE {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    ring_tie(fa);
    ring_tie(fb);
  };
  // One k-step: the products of (fa, fb); behind every other one a fragment read of the NEXT k-step into (na, nb),
  // and NL tile loads, evenly spaced, into the slot at byte offset `slot`.  hook(m): what else is to stand behind product m.
  auto kstep = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[JT], ring_u32x4 (&na)[FI], ring_u32x4 (&nb)[JT], uint32_t ab, uint32_t bb,
                   auto IS_A, const char* base, uint32_t slot, auto&& hook) DLLAVA_INLINE {
    constexpr int NL = decltype(IS_A)::value ? FI : JT;
    constexpr int kGap = kMF / NL;
    static_for<kMF>([&](auto Mi) DLLAVA_INLINE {
      constexpr int m = decltype(Mi)::value;
      ring_mfma(acc[m / JT][m % JT], fa[m / JT], fb[m % JT]);
      if constexpr (m % 2 == 0 && m / 2 < kNR) read1(na, nb, ab, bb, std::integral_constant<int, m / 2>{});
      if constexpr (m % kGap == kGap - 1 && m / kGap < NL) {
        if constexpr (decltype(IS_A)::value)
          dma(base + ga[m / kGap], slot, m / kGap);
        else
          dma(base + gb[m / kGap], slot, m / kGap);
      }
      hook(std::integral_constant<int, kMF - 1 - m>{});
      if constexpr (m % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    });
  };
  static_assert(kMF / 2 >= kNR, "a k-step has room for the reads of the next one");

  // Half-stages in ring order: h(2k) = B of stage k, h(2k+1) = A of stage k; h(n) lives in slot n % 5.
  // Iteration k multiplies stage k.  Behind its first k-step it requests B(k+2) into the slot of A(k-1), behind its
  // second -- after its barrier -- A(k+2) into stage k's own B slot.  The barrier needs A(k+1) and B(k+1): everything
  // but the JT loads of B(k+2).
  constexpr uint32_t kS = 32 * FI * kRingRowBytes;
  static_for<JT>([&](auto J) DLLAVA_INLINE { dma(Bbase + koff(0) + gb[J.value], 0 * kS, J.value); });
  static_for<FI>([&](auto J) DLLAVA_INLINE { dma(Abase + koff(0) + ga[J.value], 1 * kS, J.value); });
  static_for<JT>([&](auto J) DLLAVA_INLINE { dma(Bbase + koff(1) + gb[J.value], 2 * kS, J.value); });
  static_for<FI>([&](auto J) DLLAVA_INLINE { dma(Abase + koff(1) + ga[J.value], 3 * kS, J.value); });
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(JT + FI) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("s_nop 15" ::: "memory");  // the accumulators' first values, written by plain instructions, before the first product
  static_for<kNR>([&](auto I) DLLAVA_INLINE { read1(ua, ub, a_at + kS, b_at, I); });

  const char* Ak = Abase + koff(2);  // stage kt + 2 of either matrix
  const char* Bk = Bbase + koff(2);
  uint32_t o0 = 0, o1 = kS, o2 = 2 * kS, o3 = 3 * kS, o4 = 4 * kS;  // byte offsets of the slots of B(k), A(k), B(k+1), A(k+1), B(k+2)
  uint32_t ab = (a_at ^ 64u) + o1, bb = (b_at ^ 64u) + o0;
  int left = nk;  // stages still to multiply
  do {
    wait(ua, ub);
    kstep(ua, ub, va, vb, ab, bb, std::false_type{}, Bk, o4, [&](auto E) DLLAVA_INLINE {
      if constexpr (decltype(E)::value == 4) {
        ab = a_at + o3;
        bb = b_at + o2;
      }
    });
    // the fragments of the last k-step are in registers: this wave is done with the stage's slots
    wait(va, vb);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(JT) : "memory");
    __builtin_amdgcn_s_barrier();
    kstep(va, vb, ua, ub, ab, bb, std::true_type{}, Ak, o0, [&](auto E) DLLAVA_INLINE {
      if constexpr (decltype(E)::value == 6) {
        if (left > 3) {
          Ak += kRingBK * 2;
          Bk += kRingBK * 2;
        }
      }
      if constexpr (decltype(E)::value == 4) {
        const uint32_t t0 = o0, t1 = o1;
        o0 = o2, o1 = o3, o2 = o4, o3 = t0, o4 = t1;
      }
      if constexpr (decltype(E)::value == 2) {
        ab = (a_at ^ 64u) + o1;
        bb = (b_at ^ 64u) + o0;
      }
    });
  } while (--left > 0);
  // the reads and loads issued for stages past the end are drained, and the last products (whose latency the
  // compiler does not know) have been written
  wait(ua, ub);
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  static_for<FI>([&](auto I) DLLAVA_INLINE { static_for<JT>([&](auto J) DLLAVA_INLINE { ring_tie_acc(acc[I.value][J.value]); }); });
}

// 32*FI x 32*TJ x d tile product for launches whose tiles of 256 rows would leave most of the chip idle: the same wave
// layout (2 x 2 waves, wave w: A rows 16*FI*(w/2), B rows 16*TJ*(w%2)), fragments and LDS row layout as above.
// Such a tile is bound by the bytes its compute unit pulls (32 KiB per stage at 128 x 128 against 0.25 us of products)
// and by their latency, so the block's share of the LDS (all of it, half or a third) is a ring of D whole stages: a stage's
// slot is requested again, D stages ahead, once its last fragments are in registers.  A wave issues in order and stalls on
// loads issued together, so the loads are dealt out, unconditionally, behind the products of a whole stage (128 x 128: 0.44 us
// a stage with all of them at its end, 0.37 us dealt out; 0.62 us in the two-slot form with staging registers that this
// replaced; under a condition each, the compiler moved the accumulators out of their registers and back).  One barrier per
// stage, before its last k-step.
// Register r of acc[i][j]: A row 16*FI*(w/2) + 16*i + 4*(lane/16) + r  .  B row 16*TJ*(w%2) + 16*j + lane%16.
// As above: clamped rows, all LDS traffic complete on return, a block barrier before the memory is used for something else.
template <int FI, int TJ, int D>
__device__ __forceinline__ void gemm_ring_small(const char* Abase, const int64_t (&ga)[FI], const char* Bbase, const int64_t (&gb)[TJ],
                                                int nk, DLLAVA_LDS char* smem, int w, ring_f32x4 (&acc)[FI][TJ]) {
  constexpr int kMF = FI * TJ, kNR = FI + TJ, kL = FI + TJ;  // products and fragment reads per k-step, tile loads per stage
  constexpr int kL1 = kL / 2;  // loads behind the stage's last k-step; the others follow behind the next stage's first
  constexpr uint32_t kA = 32 * FI * kRingRowBytes, kS = kA + 32 * TJ * kRingRowBytes;  // bytes of a stage's A part, of a stage
  static_assert(D >= 3 && (D - 1) * kL < 64, "the wait counter holds the loads in flight");
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t s0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t fo = (lane & 15) * kRingRowBytes + (((lane >> 4) ^ ((lane & 15) >> 1)) * 16);
  const uint32_t a_at = s0 + (w >> 1) * (16 * FI) * kRingRowBytes + fo, b_at = s0 + kA + (w & 1) * (16 * TJ) * kRingRowBytes + fo;
  ring_u32x4 ua[FI], ub[TJ], va[FI], vb[TJ];

  auto dma1 = [&](int64_t k, uint32_t slot, auto I) DLLAVA_INLINE {
    constexpr int i = decltype(I)::value;
    const char* src = i < FI ? Abase + k + ga[i < FI ? i : 0] : Bbase + k + gb[i < FI ? 0 : i - FI];
    const uint32_t at = slot + (i < FI ? 0 : kA) + (w + 4 * (i < FI ? i : i - FI)) * 1024;
    __builtin_amdgcn_global_load_lds((const DLLAVA_GLB void*)src, (DLLAVA_LDS void*)(smem + at), 16, 0, 0);
  };
  auto read1 = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[TJ], uint32_t ab, uint32_t bb, auto I) DLLAVA_INLINE {
    constexpr int i = decltype(I)::value;
    if constexpr (i < FI)
      fa[i] = ring_lds_read16<i * 16 * kRingRowBytes>(ab);
    else
      fb[i - FI] = ring_lds_read16<(i - FI) * 16 * kRingRowBytes>(bb);
  };
  auto wait = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[TJ]) DLLAVA_INLINE {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    ring_tie(fa);
    ring_tie(fb);
  };
  // the products of (fa, fb); behind them the reads of the next k-step and loads L0 .. L0+NL-1 of a stage
  auto kstep = [&](ring_u32x4 (&fa)[FI], ring_u32x4 (&fb)[TJ], ring_u32x4 (&na)[FI], ring_u32x4 (&nb)[TJ], uint32_t ab, uint32_t bb,
                   auto L0, auto NL, int64_t k, uint32_t slot) DLLAVA_INLINE {
    static_for<kMF>([&](auto Mi) DLLAVA_INLINE {
      constexpr int m = decltype(Mi)::value, n = decltype(NL)::value;
      ring_mfma(acc[m / TJ][m % TJ], fa[m / TJ], fb[m % TJ]);
      if constexpr (m < kNR) read1(na, nb, ab, bb, Mi);
      constexpr int i = m * n / kMF;  // load i stands behind the last product with that quotient
      if constexpr (i != (m + 1) * n / kMF)
        dma1(k, slot, std::integral_constant<int, decltype(L0)::value + i>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  static_assert(kMF >= kNR && kMF >= kL - kL1, "a k-step has room for the reads of the next one");
  // byte offset along d of stage k; stages past the end re-read the last one (in bounds, unused)
  auto koff = [&](int k) DLLAVA_INLINE { return static_cast<int64_t>(k < nk ? k : nk - 1) * (kRingBK * 2); };
  // Loads are counted: stage k + D's follow stage k's barrier, the first kL1 behind its last k-step, the others behind the
  // next stage's first.
  static_for<D - 1>([&](auto P) DLLAVA_INLINE { static_for<kL>([&](auto I) DLLAVA_INLINE { dma1(koff(P.value), P.value * kS, I); }); });
  static_for<kL1>([&](auto I) DLLAVA_INLINE { dma1(koff(D - 1), (D - 1) * kS, I); });
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2) * kL + kL1) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("s_nop 15" ::: "memory");  // the accumulators' first values, written by plain instructions, before the first product
  static_for<kNR>([&](auto I) DLLAVA_INLINE { read1(ua, ub, a_at, b_at, I); });
  uint32_t here = 0, before = (D - 1) * kS;  // byte offsets of the slots of this stage and of the one before it
  int64_t ahead = koff(D - 1);               // of the stage that goes into slot `before`
  for (int k = 0; k < nk; ++k) {
    wait(ua, ub);
    kstep(ua, ub, va, vb, (a_at ^ 64u) + here, (b_at ^ 64u) + here, std::integral_constant<int, kL1>{},
          std::integral_constant<int, kL - kL1>{}, ahead, before);
    // the fragments of the last k-step are in registers: this wave is done with the stage's slot
    wait(va, vb);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2) * kL) : "memory");  // stage k + 1 has landed
    __builtin_amdgcn_s_barrier();
    before = here;
    here = here + kS < D * kS ? here + kS : 0;
    ahead = koff(k + D);
    kstep(va, vb, ua, ub, a_at + here, b_at + here, std::integral_constant<int, 0>{}, std::integral_constant<int, kL1>{}, ahead, before);
  }
  wait(ua, ub);  // reads and loads issued for stages past the end are drained
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");  // the last products, whose latency the compiler does not know, are written
  static_for<FI>([&](auto I) DLLAVA_INLINE { static_for<TJ>([&](auto J) DLLAVA_INLINE { ring_tie_acc(acc[I.value][J.value]); }); });
}

}  // namespace dllava
