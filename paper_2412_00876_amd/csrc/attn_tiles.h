// Attention of whole sequences on the matrix cores, bfloat16: the body of the kernels of prefill_tiles.hip (causal over the
// kept rows, Eq. 1 of the paper applied to S^{P*}, keys and values in pages or in rows; unmasked within spans) and masked_mfma.hip
// (the training form, Eq. 7: the keep mask inside the softmax, over the full token set).
//
// One work item is (sequence, head, NWQ*32 consecutive query rows), served by a block of NWQ waves of 32 queries that walks
// the key tiles (32 keys) up to its diagonal.  K and V tiles go from global memory straight into rings of three LDS buffers
// each (asynchronous loads, two tiles ahead of their use, K one tile before V; one block barrier per tile).
//
// The score tile is computed TRANSPOSED, S^T = K Q^T (keys down the rows, queries across the columns) with
// v_mfma_f32_32x32x16_bf16.  In the result layout a lane then holds 16 keys of ONE query (its partner lane l^32 holds the
// other 16), and the probabilities are already laid out as the B operand of the second product O^T = V^T P^T: they are split
// in place into two bfloat16 operands (16 significant bits) and never leave registers.  The contraction order of that second
// product is chosen to match the order in which S^T leaves the keys in a lane; V stays row-major ([key][dim]) in LDS and the
// matching A fragments (four consecutive keys of one dim per lane) come from the transposing LDS read.
//
// What bounds it.  Per tile of a wave at head size 128: 24 products of 32 clocks (768), and 137 issue slots of 4 clocks for
// the softmax (per score a multiplication, an exponential of two slots, three to split it and half of two packs, an addition,
// half a maximum).  Beside one 32x32x16 product six vector slots are free (measured: a product and six plain instructions 34.7
// clocks with two waves per SIMD, 43 with eight); beside a 16x16x32 product of half the size two (17.3; with three 21.3), so
// the larger product hides half as much again.  The tile step is therefore software-pipelined over the key tiles of ONE group
// of 32 queries, about six vector instructions behind each product, pinned there by scheduling barriers:
//     tile t:  softmax(t)  beside  P(t-1) V, K Q(t+1)
// From LDS alone (no loads, no barrier) it takes 906 clocks per tile and SIMD; at that rate the power limit leaves 1.5 GHz, 600 ns.
// In the whole kernel a tile takes 770 ns at 1.9 GHz; in copies of it without one part each, the tiles' loads cost 13 %, the
// arithmetic of the next tile's addresses 4 %, the barrier 4 %, and of two blocks of a compute unit the older one is served first
// and ends at three quarters of the launch.  Where the block's part of a tile stands was measured both ways: in front of the
// products for heads of 128 (2900-row sequences 436 us, among the products 450), among them for heads of 64.
// Tried and not kept: blocks of eight waves (256 queries per K/V tile: 458 against 448 us), the loads dealt out one by one (465), items
// ordered so that a die's blocks share sequences (435 against 424 in rows).
// Measured against the forms before it (products, softmax and products one after the other; for masks two groups of 16 queries with
// 16x16x32 products): 4 sequences of 2888..3085 rows, 32 heads of 128, pages 500 -> 428 us; 16 of 158..355 rows 43.3 -> 38.2;
// masked, 8 of 619..816 rows 111 -> 84; unmasked, 4 spans of 2880, 8 heads of 64 138 -> 120.
//
// With masks the work is the visible keys, not all keys: in front of an item's own 128 rows a key is either visible to all of its
// queries or to none, so those keys come from a list of the visible ones (prefill_args.h), 32 at a time, and such a tile needs no
// mask; only the item's own rows are walked as they stand, under the mask words.  A row's place is a scalar load, dealt to the lanes
// that fetch the row.  Where the visible keys fill the tiles that have any (hidden tokens in long runs), those tiles are walked as they
// stand, and the tiles without a visible key are left out; their number, which the mask kernel counts, says how the item's tiles pair.
// 8 sequences of 619..816 rows, 32 heads of 128, walking all tiles / now: a fifth of the picture kept 92 / 56 us, half 92 / 69, nothing
// hidden 87 / 86; 4 of 2900..3050 461 / 156, 481 / 275, 468 / 447, of five pictures of 576 rows three visible 312 / 301 (walking the tiles with a
// visible key / now); heads of 64 303 / 92, 306 / 166, 282 / 271, 196 / 185.
// The stream of tile loads meets every tile first, so it hands the tiles' masks on (mask0..2); what an item needs once is read
// from the kernel's arguments each time.  With those kept and the masks found twice 29 to 47 scalar registers were spilled, now none.
#pragma once

#include <atomic>
#include <type_traits>

#include "gemm_ring.h"
#include "prefill_args.h"

namespace dllava {

namespace {  // internal to each source that includes this

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // native vector: always promoted to registers

constexpr int kBN = 32;  // keys per tile

// The lane number, found where it is needed: kept, it would take a register across the tile loop.
__device__ __forceinline__ int lane_here() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\ts_nop 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// One wave-wide load straight into LDS: 16 bytes per lane from base + offset to lds_addr + 16*lane (wave-uniform base and
// lds_addr).  Written as an instruction for its scalar base: the compiler adds the base in every lane.  The base has passed
// through base_ready() since it was computed.
__device__ __forceinline__ uint32_t lds_address(bf16_t* p) { return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)p)); }
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t offset, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds_addr) : "memory");
}
// A scalar register that a vector instruction has written (a lane's value made uniform) may be a load's base five wait states later.
__device__ __forceinline__ void base_ready(const char*& lo, const char*& hi) { asm volatile("s_nop 4" : "+s"(lo), "+s"(hi)); }
// the same from an address per lane (M0, the LDS address of such loads, is set by these two statements only)
__device__ __forceinline__ void load_to_lds(const char* src, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory");
}

// Tile staging.  K and V rows of a key tile go from global memory straight into LDS (no registers in between):
// a wave-wide 16-byte load deposits its 64 pieces at consecutive LDS addresses, i.e. 1 KiB = 64/(DH/8) whole rows,
// so a tile is row-major without padding and bank conflicts are avoided by permuting the 16-byte chunks of a row
// on the way in (the lane that fills physical chunk pc of tile row rr fetches logical chunk pc ^ f(rr)):
//   K (and the queries): f(rr) = rr mod 16 (rows of 256 bytes), (rr/2) mod 8 (rows of 128 bytes).  The 16 lanes that read
//      one logical chunk of 16 different rows hit 16 different bank groups.
//   V: f(rr) = 4*(rr mod chunks/4).   V is read with the transposing LDS load (4 keys x 16 dims per 16 lanes); the
//      4 keys of such a read then lie in 4 different 64-byte bank groups.
// Rows past the last needed key repeat it (lim = last_key - t*kBN): the causal test masks them, but they must
// hold finite data, which unwritten page slots need not.
template <int DH, int NWQ>
struct Dma {
  static constexpr int kChunks = DH / 8;            // 16-byte chunks per row
  static __device__ __forceinline__ int k_swizzle(int rr) { return DH == 128 ? rr % 16 : (rr >> 1) % 8; }
  static constexpr int kRowsPerLoad = kWave / kChunks;
  static constexpr int kLoads = kBN / (kRowsPerLoad * NWQ);  // wave-wide loads per wave per tile, for K and again for V
  static_assert(kLoads >= 1 && kLoads * kRowsPerLoad * NWQ == kBN, "tile does not divide among the waves");
};

// The running maximum is only a reference point of the exponentials: any value within a few powers of two of the
// true maximum serves.  The accumulators are rescaled only when some query's tile maximum exceeds its reference by
// more than this many powers of two (probabilities then stay below 2^kSlack; their bfloat16 split is relative, so
// nothing is lost), which after the first tile of a sequence is rare.
constexpr float kSlack = 8.f;
constexpr float kNoReference = -1e30f;  // finite floor, not -inf: a query that sees no key of the first tiles keeps its state

// LDS reads of the tiles are written as instructions: the compiler would otherwise order every LDS read after ALL
// outstanding asynchronous fills (it cannot tell the buffers apart) and so wait for the tiles just requested.
// The reads return in order; the fragments pass through the statement that waits for them.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int OFF>
__device__ __forceinline__ u32x2 lds_read8_tr16(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_read16_acc(uint32_t addr) {  // into accumulation registers
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=a"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void tie4_acc(u32x4& v) { asm volatile("" : "+a"(v)); }
__device__ __forceinline__ void tie2(u32x2& v) { asm volatile("" : "+v"(v)); }
// The products, with the operand files chosen here: scores, probabilities and V in vector registers, outputs, queries and K
// in accumulation registers.
__device__ __forceinline__ void qk_first(f32x16& s, const u32x4& k, const u32x4& q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "a"(k), "a"(q));
}
__device__ __forceinline__ void qk_next(f32x16& s, const u32x4& k, const u32x4& q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(k), "a"(q));
}
__device__ __forceinline__ void pv(f32x16& o, const u32x4& v, const u32x4& p) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(v), "v"(p));
}
__device__ __forceinline__ void products_done() { asm volatile("s_nop 15\n\ts_nop 3" ::: "memory"); }
__device__ __forceinline__ void tie_s(f32x16& s) { asm volatile("" : "+v"(s)); }
__device__ __forceinline__ void tie_o(f32x16& o) { asm volatile("" : "+a"(o)); }
// zeros written where they belong (as a constant the compiler keeps a vector of them for the whole loop)
__device__ __forceinline__ void zero_o(f32x16& o) {
  static_for<16>([&](auto I) DLLAVA_INLINE {
    float z;
    asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(z));
    o[I.value] = z;
  });
  tie_o(o);
}

// Scalars dealt to the lanes, v[i] to the i-th fourth or eighth of the wave: a plain move each, under a mask of lanes that walks
// through the wave.  (As selections between the scalars, each of which takes a vector register first, it is twice the
// instructions.)  All lanes are active.
__device__ __forceinline__ uint32_t by_lanes(const uint32_t (&v)[4]) {
  uint32_t r;
  uint64_t all;
  asm volatile(
      "s_mov_b64 %1, exec\n\ts_mov_b64 exec, 0xffff\n\tv_mov_b32 %0, %2\n\ts_lshl_b64 exec, exec, 16\n\tv_mov_b32 %0, %3\n\t"
      "s_lshl_b64 exec, exec, 16\n\tv_mov_b32 %0, %4\n\ts_lshl_b64 exec, exec, 16\n\tv_mov_b32 %0, %5\n\ts_mov_b64 exec, %1"
      : "=&v"(r), "=&s"(all)
      : "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3])
      : "scc");
  return r;
}
__device__ __forceinline__ uint32_t by_lanes(const uint32_t (&v)[8]) {
  uint32_t r;
  uint64_t all;
  asm volatile(
      "s_mov_b64 %1, exec\n\ts_mov_b64 exec, 0xff\n\tv_mov_b32 %0, %2\n\ts_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %3\n\t"
      "s_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %4\n\ts_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %5\n\t"
      "s_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %6\n\ts_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %7\n\t"
      "s_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %8\n\ts_lshl_b64 exec, exec, 8\n\tv_mov_b32 %0, %9\n\ts_mov_b64 exec, %1"
      : "=&v"(r), "=&s"(all)
      : "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7])
      : "scc");
  return r;
}

__device__ __forceinline__ float select_bits(uint32_t m, float a, float b) {  // a where m has ones, else b
  float r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(a), "v"(b));
  return r;
}

// A value passes through here where it is to be computed: the compiler otherwise moves plain arithmetic down to its use,
// out of the shadow of the products it is written beside.
__device__ __forceinline__ void here(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void here(uint32_t& x) { asm volatile("" : "+v"(x)); }
// maxima of scores as instructions: fmaxf of a value whose origin the compiler does not know costs a second instruction
__device__ __forceinline__ float max2(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// A wave's state over the tiles of an item.
template <int DH>
struct State {
  f32x16 o[DH / 32];        // outputs [32-dim block]
  u32x4 q[DH / 16];         // queries [16-dim step]
  u32x4 k[DH / 16];         // K fragments of a tile [16-dim step]
  u32x2 v[DH / 32][2][2];   // V fragments of a tile [32-dim block][16-key half]
  float m_ref, l_run;       // reference of the exponentials (in powers of two), sum of this lane's probabilities
  float thr;                // scaled score above which the reference moves; while it moves, what the outputs are multiplied with
};
struct Probs {
  u32x4 hi[2], lo[2];       // [16-key half]: B operands of the second product
};
__device__ __forceinline__ u32x4 join(const u32x2& a, const u32x2& b) { return u32x4{a[0], a[1], b[0], b[1]}; }

// Where the softmax's vector instructions stand: four stages per pair of scores, each behind the stage before it; at[i]: the
// product, of `all`, that the i-th of them stands behind.  The probabilities of the two 16-key halves (stages 2 and 3 of pairs
// 0..3 and 4..7) take the place of those of the tile before, whose last products are number half0 - 1 and half1 - 1.
struct Places {
  int stage[32], pair[32], at[32];
};
constexpr Places make_places(int first, int all, int half0, int half1) {
  Places r{};
  constexpr int w[4] = {2, 4, 3, 5};  // issue slots of a stage
  int n = 0, slots = 0;
  for (int pass = 0; pass < 4; pass += 2)
    for (int s = 0; s < 8 + 1; ++s)
      for (int st = pass + 1; st >= pass; --st) {
        const int p = s - (st - pass);
        if (p < 0 || p > 7) continue;
        int at = all > first ? first + slots * (all - first) / 112 : first;
        const int least = st < 2 ? 0 : (p < 4 ? half0 : half1);
        if (all > first && at < least) at = least < all ? least : all - 1;
        r.stage[n] = st, r.pair[n] = p, r.at[n] = at;
        slots += w[st];
        ++n;
      }
  return r;
}

// A query's maximum over its two lanes becomes the reference of the exponentials; T.thr holds the outputs' factor until
// reference_moved().
template <int DH>
__device__ __forceinline__ void move_reference(State<DH>& T, float x) {  // x: the lane's largest scaled score
  const float m_t = max2(x, __shfl_xor(x, 32, kWave));
  const float m_new = max2(T.m_ref, m_t);
  T.thr = __builtin_amdgcn_exp2f(T.m_ref - m_new);
  T.m_ref = m_new;
  T.l_run *= T.thr;
}
template <int DH>
__device__ __forceinline__ void reference_moved(State<DH>& T) { T.thr = T.m_ref + kSlack; }
__device__ __forceinline__ float max16(const f32x16& S) {
  const float x = max3(max3(S[0], S[1], S[2]), max3(S[3], S[4], S[5]), S[6]), y = max3(max3(S[7], S[8], S[9]), max3(S[10], S[11], S[12]), S[13]);
  return max3(max2(x, y), S[14], S[15]);
}
template <int DH>
__device__ __forceinline__ void first_reference(State<DH>& T, const f32x16& S, float scale_log2) {
  move_reference(T, max16(S) * scale_log2);
  reference_moved(T);
}

// Tile t of a wave: the softmax of its scores S into P, beside the products P(t-1) V (PV) and K Q of the next tile (QK, into
// Sn); V(t) is read for the next call.  The block's part of a tile -- open() (the tiles read here have landed), request_v() and
// request_k() (of later tiles) -- is called among the products, mask(S) once the scores have been written.
// kb / vb, set by open(): LDS addresses of this lane's pieces of K(t+1) and V(t).
// FIRST: the item's first tile (no P(t-1), the reference still at its floor).
template <int DH, bool FIRST, bool QK, typename Open, typename Mask, typename RequestV, typename RequestK>
__device__ __forceinline__ void step(State<DH>& T, f32x16& S, f32x16& Sn, Probs& P, const uint32_t& kb, const uint32_t& vb, float scale_log2,
                                     Open&& open, Mask&& mask, RequestV&& request_v, RequestK&& request_k) {
  constexpr int kNB = DH / 32, kKS = DH / 16, kRowBytes = DH * 2;
  constexpr int kNP = FIRST ? 0 : kNB * 4, kNQ = QK ? kKS : 0, kNM = kNP + kNQ;
  constexpr int kHead = FIRST ? 0 : 5;       // products in front of the probabilities
  constexpr bool kUpFront = DH == 128;       // open and request in front of the products
  constexpr int kReadK = kUpFront ? 0 : 2, kRequest = 4;  // products behind which K is read (two pieces each), requests are made
  constexpr int kHaveK = DH == 128 ? 9 : 6;  // K has been read
  auto read_k = [&](auto I) DLLAVA_INLINE { T.k[I.value] = lds_read16_acc<0>(kb ^ (I.value * 32)); };
  auto read_v = [&](auto I) DLLAVA_INLINE {  // piece I of 4*kNB, ordered half, block, 8-key part
    constexpr int half = I.value / (2 * kNB), nb = (I.value / 2) % kNB, part = I.value % 2;
    T.v[nb][half][part] = lds_read8_tr16<(16 * half + 8 * part) * kRowBytes>(vb ^ (nb * 64));
  };
  auto k_here = [&]() DLLAVA_INLINE {
    lds_wait();
    static_for<kKS>([&](auto I) DLLAVA_INLINE { tie4_acc(T.k[I.value]); });
  };
  auto product = [&](auto Mi) DLLAVA_INLINE {
    constexpr int m = decltype(Mi)::value;
    if constexpr (m < kNP) {
      constexpr int half = m / (2 * kNB), nb = (m / 2) % kNB;
      pv(T.o[nb], join(T.v[nb][half][0], T.v[nb][half][1]), m % 2 == 0 ? P.hi[half] : P.lo[half]);
      if constexpr (!kUpFront && m == kReadK - 1) open();
      if constexpr (QK && m >= kReadK && m < kReadK + kKS / 2) {
        read_k(std::integral_constant<int, 2 * (m - kReadK)>{});
        read_k(std::integral_constant<int, 2 * (m - kReadK) + 1>{});
      }
      if constexpr (QK && m == kHaveK) k_here();
      if constexpr (m > kHaveK - (DH == 64) && m <= kHaveK - (DH == 64) + kNB) {  // V's first half is used up
        constexpr int i = 2 * (m - kHaveK + (DH == 64) - 1);
        read_v(std::integral_constant<int, i>{});
        read_v(std::integral_constant<int, i + 1>{});
      }
    } else {
      constexpr int ks = m - kNP;
      if constexpr (ks == 0) qk_first(Sn, T.k[0], T.q[0]); else qk_next(Sn, T.k[ks], T.q[ks]);
      if constexpr (FIRST) {
        read_v(std::integral_constant<int, 4 * ks * kNB / kKS>{});
        read_v(std::integral_constant<int, 4 * ks * kNB / kKS + 1>{});
      } else if constexpr (ks >= 1 && ks <= kNB) {
        read_v(std::integral_constant<int, 2 * kNB + 2 * (ks - 1)>{});
        read_v(std::integral_constant<int, 2 * kNB + 2 * (ks - 1) + 1>{});
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!FIRST && !kUpFront && m == kRequest) request_v();
    if constexpr (!FIRST && !kUpFront && m == kRequest + 1) request_k();
    if constexpr (!FIRST && !kUpFront && (m == kRequest || m == kRequest + 1)) __builtin_amdgcn_sched_barrier(0);
  };
  float x, y, z, w;
  auto max_a = [&]() DLLAVA_INLINE {
    x = max3(S[0], S[1], S[2]), y = max3(S[3], S[4], S[5]), z = max3(S[6], S[7], S[8]), w = max3(S[9], S[10], S[11]);
    here(x), here(y), here(z), here(w);
  };
  auto max_b = [&]() DLLAVA_INLINE {
    x = max3(x, y, S[12]), z = max3(z, w, S[13]);
    x = max3(x, S[14], S[15]);
    x = max2(x, z);
    here(x);
  };
  if constexpr (FIRST || kUpFront) open();
  if constexpr (FIRST && QK) static_for<kKS>(read_k);
  if constexpr (FIRST || kUpFront) {
    request_v();
    request_k();
  }
  if constexpr (FIRST) {
    products_done();
    tie_s(S);
    mask(S);
    max_a();
    max_b();
    if constexpr (QK) k_here();
  } else {
    // the maximum stands behind the fourth product: the scores' own last product must have been written
    static_for<kHead>([&](auto Mi) DLLAVA_INLINE {
      product(Mi);
      if constexpr (decltype(Mi)::value == 3) {
        mask(S);
        max_a();
      }
      if constexpr (decltype(Mi)::value == 4) max_b();
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  // The two lanes of a query look at their own scores only; the maximum itself is needed when one of them is past the threshold.
  // (Scaled before it is compared, as in the kernel for short sequences: the reference then moves at the same scores there and here.)
  x *= scale_log2;
  bool moved = false;
  if constexpr (FIRST) {  // neither the threshold nor a factor takes a register before the end of the tile
    if (__any(x > kNoReference + kSlack)) T.m_ref = max2(T.m_ref, max2(x, __shfl_xor(x, 32, kWave)));
  } else if (__any(x > T.thr)) {
    move_reference(T, x);
    moved = true;
  }
  constexpr Places places = make_places(kHead, kNM, kNP / 2 + 1, kNP + 1);
  float p0[8], p1[8], a0[8], a1[8], sum;
  auto op = [&](auto Oi) DLLAVA_INLINE {
    constexpr int st = places.stage[decltype(Oi)::value], p = places.pair[decltype(Oi)::value];
    if constexpr (st == 0) {
      p0[p] = __builtin_fmaf(S[2 * p], scale_log2, -T.m_ref);
      p1[p] = __builtin_fmaf(S[2 * p + 1], scale_log2, -T.m_ref);
      here(p0[p]), here(p1[p]);
    } else if constexpr (st == 1) {
      p0[p] = __builtin_amdgcn_exp2f(p0[p]);
      p1[p] = __builtin_amdgcn_exp2f(p1[p]);
      here(p0[p]), here(p1[p]);
    } else if constexpr (st == 2) {
      uint32_t h = __builtin_amdgcn_perm(__float_as_uint(p1[p]), __float_as_uint(p0[p]), 0x07060302u);  // {hi16(p0), hi16(p1)}
      here(h);
      P.hi[p / 4][p % 4] = h;
      a0[p] = __uint_as_float(__float_as_uint(p0[p]) & 0xffff0000u);
      a1[p] = __uint_as_float(__float_as_uint(p1[p]) & 0xffff0000u);
      here(a0[p]), here(a1[p]);
    } else {
      const float r0 = p0[p] - a0[p], r1 = p1[p] - a1[p];
      // the tile's probabilities are added up among themselves, pair by pair, before they join the sum of the tiles: a long row of
      // single additions to that sum loses more of it, and these are the sums of the kernel for short sequences, bit for bit
      const float pair = p0[p] + p1[p];
      uint32_t l = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
      here(l);
      P.lo[p / 4][p % 4] = l;
      sum = p == 0 ? pair : sum + pair;
      if constexpr (p == 7) T.l_run += sum;
      here(p == 7 ? T.l_run : sum);
    }
  };
  static_for<(kNM - kHead > 0 ? kNM - kHead : 1)>([&](auto Ri) DLLAVA_INLINE {
    constexpr int i = decltype(Ri)::value;
    if constexpr (kNM > kHead) product(std::integral_constant<int, kHead + i>{});
    static_for<32>([&](auto Oi) DLLAVA_INLINE {
      if constexpr (places.at[decltype(Oi)::value] == kHead + i) op(Oi);
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  if constexpr (!QK) {  // V's rest: there was no product of K Q to read it behind
    constexpr int from = FIRST ? 0 : 2 * kNB;
    if constexpr (!FIRST) asm volatile("s_nop 7" ::: "memory");
    static_for<4 * kNB - from>([&](auto I) DLLAVA_INLINE { read_v(std::integral_constant<int, from + decltype(I)::value>{}); });
  }
  if constexpr (FIRST) {
    reference_moved(T);
  } else if (moved) {  // P(t-1) V went in under the old reference
    products_done();
    static_for<kNB>([&](auto I) DLLAVA_INLINE {
      tie_o(T.o[I.value]);
      T.o[I.value] *= T.thr;
      tie_o(T.o[I.value]);
    });
    reference_moved(T);
  }
  lds_wait();
  static_for<4 * kNB>([&](auto I) DLLAVA_INLINE { tie2(T.v[I.value % kNB][(I.value / (2 * kNB))][(I.value / kNB) % 2]); });
}

// The last P V of an item.
template <int DH>
__device__ __forceinline__ void finish(State<DH>& T, const Probs& P) {
  constexpr int kNB = DH / 32;
  asm volatile("s_nop 1" ::: "memory");  // plain writes of the outputs or the probabilities before a product
  static_for<4 * kNB>([&](auto Mi) DLLAVA_INLINE {
    constexpr int m = decltype(Mi)::value, half = m / (2 * kNB), nb = (m / 2) % kNB;
    pv(T.o[nb], join(T.v[nb][half][0], T.v[nb][half][1]), m % 2 == 0 ? P.hi[half] : P.lo[half]);
  });
  products_done();
  static_for<kNB>([&](auto I) DLLAVA_INLINE { tie_o(T.o[I.value]); });
}

// Paged: causal, keys and values in the cache's pages.  Rows: causal, in rows.  Full: every query sees all keys of its sequence.
// Masked: causal, keys hidden by key words but from their own query.  Words: the same without counts and list of the visible keys.
enum class Mode { Paged, Rows, Full, Masked, Words };

// One work item = (sequence, head, tile of NWQ*32 query rows).  Blocks are PERSISTENT: the launch holds as many blocks as
// fit the chip at once (slots), block p takes every slots-th item and walks their key tiles as ONE stream: the tile
// loads run two tiles ahead of the arithmetic across item boundaries, and the queries of the next item go to LDS while
// the current item runs.  A block that starts needs three or four dependent trips to memory before its first tile; a
// persistent block pays them once.
// Items are numbered by DESCENDING query-tile index over all sequences, heads adjacent: a causal item's work grows
// with its tile index, so every block takes its longest items first and the launch ends with the shortest ones.
template <int DH, int NWQ, Mode MODE>
__device__ __forceinline__ void attend_items(const PrefillArgs& args) {
  constexpr bool kFull = MODE == Mode::Full, kList = MODE == Mode::Masked, kMasks = kList || MODE == Mode::Words;
  // the arguments as locals (the closures below then capture plain values, which the compiler keeps in registers)
  const int aB = args.B;
  const float aScale = args.scale_log2;
  const void* const aK = args.K;
  const void* const aV = args.V;
  // What is needed once an item is, with masks, read from the arguments each time (`args` is the kernel's one parameter): kept, it would
  // cost spills of scalar registers.
  typedef const PrefillArgs __attribute__((address_space(4)))* ConstArgs;
  auto arg = [&](auto field) DLLAVA_INLINE {
    if constexpr (kMasks) {
      ConstArgs p = (ConstArgs)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(p));
      return p->*field;
    } else {
      return args.*field;
    }
  };
  constexpr int kBM = NWQ * 32;
  constexpr int kChunks = DH / 8;  // 16-byte chunks per row
  constexpr int kNB = DH / 32;     // 32-dim blocks of the output
  constexpr int kKS = DH / 16;     // 16-dim steps of the first product
  constexpr int kRowBytes = DH * 2;
  constexpr int kTileElems = kBN * DH;
  constexpr int kStages = 3;
  using D = Dma<DH, NWQ>;

  // rings of three K tiles and three V tiles, and every wave's 32 queries of the block's next item (together half of a
  // compute unit's LDS at most: two blocks share it)
  __shared__ __align__(1024) bf16_t sK[kStages * kTileElems];
  __shared__ __align__(1024) bf16_t sV[kStages * kTileElems];
  __shared__ __align__(1024) bf16_t sQ[NWQ * 32 * DH];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wq = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int H = args.H;
  // Offsets, page table and mask words were written by earlier launches and do not change while this kernel runs:
  // read through the constant address space, block-uniform indices become scalar loads.  (As plain pointers they
  // may alias the output, which this kernel stores inside its loop, and every one of them would be a vector
  // load with a full vector-memory wait behind it -- a wait for the tile loads in flight.)
  typedef const int32_t __attribute__((address_space(4)))* ConstI32;
  typedef const uint32_t __attribute__((address_space(4)))* ConstU32;
  const ConstI32 off_c = (ConstI32)args.off;
  const ConstI32 bt_c = (ConstI32)args.block_table;
  const ConstU32 kw_c = (ConstU32)args.key_words;
  constexpr bool paged = MODE == Mode::Paged;
  const int step_blocks = static_cast<int>(gridDim.x);
  const uint32_t row_bytes = paged ? kRowBytes : static_cast<uint32_t>(H) * kRowBytes;

  auto uniform = [](int v) DLLAVA_INLINE { return __builtin_amdgcn_readfirstlane(v); };  // said to the compiler where it cannot see it
  // Which (sequence, query tile) is item k?  With at most 64 sequences every wave keeps the sequences' offsets in
  // its lanes (lane = sequence; one trip to memory per block) and counts with ballots; with more, the sequences are
  // walked with scalar loads (then there is one item per block).
  const bool by_lane = aB <= kWave;
  int nb_l = 0, total = 0;
  if (by_lane) {
    int off_l = lane < aB ? off_c[lane] : 0, end_l = lane < aB ? off_c[lane + 1] : 0;
    // The offsets have arrived; the statement also tells the compiler so: it would otherwise order every later use
    // of them, in loops it cannot see through, behind ALL outstanding vector-memory operations -- the tile loads.
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(off_l), "+v"(end_l));
    nb_l = (end_l - off_l + kBM - 1) / kBM;  // tiles of sequence `lane`
    int cnt = 0;
    for (int i = 0; (cnt = __builtin_popcountll(__ballot(nb_l > i))) != 0; ++i) total += cnt;
  }
  struct Item {
    int valid, b, h, tile, r0, n;
    int seen;  // with masks, in front of the item's own queries: the visible keys, which it takes from the list; or ~(tiles with a
               // visible key), which it walks
  };
  constexpr int kListPays = DH == 128 ? 11 : 16;
  auto tiles_listed = [](int seen) DLLAVA_INLINE { return static_cast<int>((static_cast<uint32_t>(seen) + kBN - 1) / kBN); };
  auto words_of = [&](const Item& it) DLLAVA_INLINE { return kw_c + ((it.r0 >> 5) + it.b); };
  auto seen_before = [&](const Item& it) DLLAVA_INLINE {
    int shown = 0;
    const int own = it.tile * (kBM / kBN);
    if constexpr (kList) {
      if (own == 0) return 0;
      const ConstU32 counts = words_of(it) + arg(&PrefillArgs::mask_slots) + own;
      const int seen = static_cast<int>(counts[0]);
      shown = static_cast<int>(counts[-1]);
      // A tile from the list takes about 1.1 times as long as one in rows whose keys are all visible (its rows' places are loads in
      // front of it; heads of 64: 1.05) and no longer than one in rows with hidden keys, whose scores pass a mask.  4 x 3000 rows, 32
      // heads, from the list / in rows: 85 % visible, scattered, 411 / 485 us (heads of 64: 251 / 308), half visible in runs of 192 on
      // average 282 / 300 (167 / 180), three of five pictures of 576 rows 316 / 301.  Short sequences: the list has to spare a tile.
      if (kListPays * tiles_listed(seen) <= (kListPays - 1) * shown && !(static_cast<uint64_t>(static_cast<uint32_t>(it.n)) * row_bytes >> 32)) return seen;
    } else if constexpr (kMasks) {
      for (int t = 0; t < own; ++t) shown += words_of(it)[t] != 0u;
    }
    return ~shown;
  };
  // Item k of a launch over at most 64 sequences.
  auto locate = [&](int k) __attribute__((always_inline)) {
    Item it{0, 0, 0, 0, 0, 0, -1};
    const int heads = arg(&PrefillArgs::H), yd = k / heads;  // position in DESCENDING tile-index order
    it.h = k - yd * heads;
    const int y = total - 1 - yd;  // position in ascending order
    if (y < 0) return it;          // (total is 0 for more sequences: those have one item per block)
    int below = 0, tile = 0;       // tiles with a smaller index
    for (;; ++tile) {
      const int cnt = __builtin_popcountll(__ballot(nb_l > tile));
      if (below + cnt > y) break;
      below += cnt;
    }
    // the (y - below)-th sequence, in ascending order, that has a tile of this index
    const unsigned long long has = __ballot(nb_l > tile);
    const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(has >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(has), 0));
    const unsigned long long me = __ballot(nb_l > tile && before == y - below);
    it.b = uniform(__builtin_ctzll(me));
    it.tile = tile;
    const ConstI32 off = (ConstI32)arg(&PrefillArgs::off) + it.b;
    it.r0 = off[0];
    it.n = off[1] - it.r0;
    it.valid = 1;
    it.seen = seen_before(it);
    return it;
  };
  // keys 0..last_key of its sequence are needed by an item
  auto last_key_of = [&](const Item& it) __attribute__((always_inline)) {
    return (!kFull && it.tile * kBM + kBM < it.n ? it.tile * kBM + kBM : it.n) - 1;
  };

  // Round j of block p takes item p + j*step, in odd rounds (step-1-p) + j*step: the rounds run through the items
  // (sorted by descending work) in alternating directions, so a block that got a longer item in one round gets a
  // shorter one in the next and the blocks' totals stay close (C5 shape: 40..42 tiles per block instead of 36..46).
  const int pblk = static_cast<int>(blockIdx.x);
  auto item_of = [&](int j) __attribute__((always_inline)) { return ((j & 1) ? step_blocks - 1 - pblk : pblk) + j * step_blocks; };
  int jC = 0;
  Item C{0, 0, 0, 0, 0, 0, -1};
  if (by_lane) {
    C = locate(item_of(0));
  } else {
    // Many sequences, one item per block: numbered sequence by sequence, the late (long) tiles of each first.  Found 64
    // sequences at a time (as a scalar walk, a chain of loads, 500 sequences of one row and 8 heads took 199 us, now 45).
    int tile = pblk / H;
    for (int b0 = 0; b0 < aB; b0 += kWave) {
      const int b = b0 + lane;
      const int r0 = b < aB ? off_c[b] : 0, n = b < aB ? off_c[b + 1] - r0 : 0;
      const int nt = (n + kBM - 1) / kBM, upto = wave_incl_scan(nt);  // tiles of the sequences up to this lane's
      const unsigned long long past = __ballot(upto > tile);
      if (past) {
        const int l = __builtin_ctzll(past);
        // the sequence's first tile is number upto - nt, its last upto - 1: counted from the last
        C = {1, b0 + l, pblk % H, __builtin_amdgcn_readlane(upto, l) - 1 - tile, __builtin_amdgcn_readlane(r0, l), __builtin_amdgcn_readlane(n, l), -1};
        C.seen = seen_before(C);
        break;
      }
      tile -= __builtin_amdgcn_readlane(upto, kWave - 1);
    }
  }
  if (!C.valid) return;

  // Which 32-query tile of an item: in every other item of a block the waves take them the other way round, so the SIMDs
  // share the longer causal tiles.  -1: none.
  auto wave_tile = [&](const Item& it, int j) DLLAVA_INLINE {
    const int t = it.tile * NWQ + ((j ^ (pblk >> 8)) & 1 ? NWQ - 1 - wq : wq);
    return it.valid && t * 32 < it.n ? t : -1;
  };
  constexpr int kQLoads = 32 / D::kRowsPerLoad;  // wave-wide loads of a wave's 32 query rows
  bf16_t* myQ = sQ + wq * 32 * DH;
  auto request_queries = [&](const Item& it, int tile, int from, int to) DLLAVA_INLINE {  // loads from .. to-1 of a wave's queries
    const int l = lane_here();
    const bf16_t* Qp = static_cast<const bf16_t*>(arg(&PrefillArgs::Q));
    const int heads = arg(&PrefillArgs::H);
    for (int i = from; i < to; ++i) {
      const int rr = D::kRowsPerLoad * i + l / kChunks, pc = l % kChunks;
      int q = (tile < 0 ? 0 : tile * 32) + rr;
      if (q >= it.n) q = it.n - 1;
      const bf16_t* src = Qp + (static_cast<size_t>(it.r0 + q) * heads + it.h) * DH + 8 * (pc ^ D::k_swizzle(rr));
      load_to_lds(reinterpret_cast<const char*>(src), lds_address(myQ) + i * (kWave * 16));
    }
  };
  // The key tiles of an item with masks: in front of its own queries the visible keys as they are listed, 32 a tile, or the tiles of the
  // sequence that have a visible key; then its own rows.  hidden(): by how many tiles these are fewer than the sequence's.
  auto hidden = [&](const Item& it) DLLAVA_INLINE {
    return kMasks ? it.tile * (kBM / kBN) - (kList && it.seen >= 0 ? tiles_listed(it.seen) : ~it.seen) : 0;
  };

  // Fragment addresses (LDS bytes, stage 0).  K: row lq, logical chunk 2*ks + g, stored at chunk ^ swizzle(lq): the
  // step ks enters as an exclusive-or with 32*ks.  Queries alike.  V: the transposing read of 16 lanes (j = lane mod 16)
  // returns to lane j four keys of dim j; lane j points at key 4*g + j/4, dims 4*(j mod 4)..+3 of the 16 dims of its
  // group; a 32-dim block enters as an exclusive-or with 64*block.
  const int g = lane >> 5, lq = lane & 31, j16 = lane & 15;
  const uint32_t k_row = lq * kRowBytes + ((g ^ D::k_swizzle(lq)) * 16);
  const uint32_t kb0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)sK)) + k_row;
  const uint32_t vb0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)sV)) +
                       (4 * g + (j16 >> 2)) * kRowBytes + ((j16 >> 2) % (kChunks / 4)) * 64 + ((lane >> 4) & 1) * 32 + (j16 & 3) * 8;

  // scores above the diagonal of some query (keys > qi), past the end of the sequence, or hidden by a zero bit of kmask (except the
  // query's own key); queries, keys and the sequence's length n as numbered by the tiles of the stream: the wave's queries are
  // those of its last tile
  auto mask_scores = [&](f32x16& S, int t, int last, int n, uint32_t kmask) DLLAVA_INLINE {
    const int j0 = t * kBN;
    if ((kFull ? j0 + kBN > n : t >= last) || (kMasks && kmask != ~0u)) {
      products_done();
      tie_s(S);
      const int l = lane_here(), g4 = 4 * (l >> 5);
      int qi = last * kBN + (l & 31);
      if (kFull || qi >= n) qi = n - 1;
      const int self = qi - j0 - g4;  // the query's own key, counted from j0 + g4
      const uint32_t upto = self < 0 ? 0u : (2u << (self < 31 ? self : 31)) - 1u;  // the keys up to it
      uint32_t seen = kMasks ? ((kmask >> g4) & upto) | (static_cast<uint32_t>(self) < 32u ? 1u << self : 0u) : upto;
      here(seen);
#pragma unroll
      for (int r = 0; r < 16; ++r) {  // key j0 + g4 + kk: two instructions each, a bit spread over a word and a selection by bits
        const int kk = 8 * (r >> 2) + (r & 3);
        const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(seen << (31 - kk)) >> 31);
        S[r] = select_bits(m, S[r], -INFINITY);
      }
    }
  };

  State<DH> T;
  auto store_item = [&](int q0, const Item& it) DLLAVA_INLINE {
    const float inv = 1.f / (T.l_run + __shfl_xor(T.l_run, 32, kWave));
    const int l = lane_here(), g = l >> 5, qi = q0 + (l & 31);
    bf16_t* orow = static_cast<bf16_t*>(arg(&PrefillArgs::O)) + (static_cast<size_t>(it.r0 + qi) * arg(&PrefillArgs::H) + it.h) * DH + 8 * g;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4 += 2) {
        // a lane holds dims 8*q4 + 4*g..+3 of a block; exchanged with its partner it holds eight consecutive dims of q4 + g
        const auto a = __builtin_amdgcn_permlane32_swap(pack_bf16x2(T.o[nb][4 * q4] * inv, T.o[nb][4 * q4 + 1] * inv),
                                                        pack_bf16x2(T.o[nb][4 * q4 + 4] * inv, T.o[nb][4 * q4 + 5] * inv), false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(pack_bf16x2(T.o[nb][4 * q4 + 2] * inv, T.o[nb][4 * q4 + 3] * inv),
                                                        pack_bf16x2(T.o[nb][4 * q4 + 6] * inv, T.o[nb][4 * q4 + 7] * inv), false, false);
        const uint4 piece = {a[0], b[0], a[1], b[1]};
        if (qi < it.n) *reinterpret_cast<uint4*>(orow + nb * 32 + 8 * q4) = piece;
      }
  };

  // ---- the stream of tile loads: item P, its tile tP is the next one whose K is requested; V follows one tile behind --------
  // A tile is two halves of 16 rows (two pages, where paged); all of a half's rows lie at fixed offsets from its first, so a
  // tile's loads are a scalar base plus a lane constant each.
  const int64_t page_half = static_cast<int64_t>(H) * kPage * kRowBytes;  // K, or V, of a page
  const int64_t v_step = paged ? page_half : static_cast<const char*>(aV) - static_cast<const char*>(aK);
  constexpr int kHalfLoads = D::kLoads >= 2 ? D::kLoads / 2 : 1;  // distinct row sets of a wave within a half
  uint32_t k_lane[kHalfLoads], v_lane[kHalfLoads];
#pragma unroll
  for (int i = 0; i < kHalfLoads; ++i) {
    const int rr = D::kRowsPerLoad * (wq + NWQ * i) + lane / kChunks, pc = lane % kChunks;
    k_lane[i] = (rr % kPage) * row_bytes + 16 * (pc ^ D::k_swizzle(rr));
    v_lane[i] = (rr % kPage) * row_bytes + 16 * (pc ^ (4 * (rr % (kChunks / 4))));
  }
  // With masks: the 16 bytes of a row that a lane fetches, the same in all its loads (their rows are a multiple of 16 apart); those of V
  // from those of K by an exclusive-or (a row's first byte is a multiple of its length).
  static_assert(!kMasks || D::kRowsPerLoad * NWQ % 16 == 0, "rows of a lane");
  auto k_chunk = [&](uint32_t l) DLLAVA_INLINE { return 16u * ((l % kChunks) ^ D::k_swizzle(D::kRowsPerLoad * wq + l / kChunks)); };
  const uint32_t v_flip = k_chunk(lane) ^ (16u * ((lane % kChunks) ^ (4 * ((D::kRowsPerLoad * wq + lane / kChunks) % (kChunks / 4)))));
  auto first_rows = [&](int i) DLLAVA_INLINE { return D::kLoads >= 2 ? i < D::kLoads / 2 : D::kRowsPerLoad * wq < kPage; };  // load i: of the first half?
  struct TileAt {
    const char *lo, *hi;  // K of the first rows of the tile's halves, this head
    int lim;              // last row of the tile that exists (>= kBN - 1: all of them)
    uint32_t k[D::kLoads];  // with masks: this lane's bytes of K, from lo (hi and lim are not used)
    uint32_t mask;          // with masks: the visible keys
  };
  int jP = 0, tP, lastP;  // lastP: its last key
  // With masks tP is the next tile in rows, or a hidden one in front of it, and wordP its mask; leftP listed keys from listP on come first.
  int leftP = 0;
  uint32_t listP = 0, wordP = 0;
  bool ended = false;  // every K tile of the block has been requested
  const char* baseP;  // K of the first row of P's sequence, its head (paged: the head's K in page 0)
  Item P = C;
  // Page ids of a tile are block-uniform scalar loads, fetched one step before the tile is requested.  The index is
  // clamped to the block table: a sequence longer than the cache capacity (flagged by the call that filled the
  // cache) then reads allocated pages, not whatever follows its row of the table.
  int pg_lo = 0, pg_hi = 0;
  auto fetch_page_ids = [&]() DLLAVA_INLINE {  // for tile tP of item P
    if (paged) {
      const ConstI32 bt = bt_c + static_cast<size_t>(P.b) * args.max_pages;
      const int last_page = lastP / kPage < args.max_pages - 1 ? lastP / kPage : args.max_pages - 1;
      pg_lo = bt[2 * tP < last_page ? 2 * tP : last_page];
      pg_hi = bt[2 * tP + 1 < last_page ? 2 * tP + 1 : last_page];
    }
  };
  auto enter = [&]() DLLAVA_INLINE {  // the stream enters item P
    P.b = uniform(P.b), P.h = uniform(P.h), P.tile = uniform(P.tile), P.r0 = uniform(P.r0), P.n = uniform(P.n);
    lastP = last_key_of(P);
    baseP = paged ? static_cast<const char*>(args.pages) + static_cast<int64_t>(P.h) * (kPage * kRowBytes)
                  : static_cast<const char*>(arg(&PrefillArgs::K)) + static_cast<int64_t>(P.r0) * row_bytes + P.h * kRowBytes;
    tP = 0;
    if constexpr (kMasks) {
      leftP = kList ? uniform(P.seen) : -1;
      if (leftP >= 0) tP = P.tile * (kBM / kBN);
      listP = 2u * static_cast<uint32_t>(arg(&PrefillArgs::mask_slots)) + static_cast<uint32_t>(P.r0) + kBN * static_cast<uint32_t>(P.b);
      wordP = words_of(P)[tP];
    }
  };
  auto next_tile_at = [&]() DLLAVA_INLINE {  // tile tP of item P; then on to the next tile of the stream
    TileAt at;
    if constexpr (kMasks) {
      if (kList && leftP > 0) {
        at.lo = baseP;
        const ConstU32 list = kw_c + listP;
#pragma unroll
        for (int i = 0; i < D::kLoads; ++i) {  // (entries past the list's end are in the workspace, too)
          uint32_t v[D::kRowsPerLoad];
#pragma unroll
          for (int e = 0; e < D::kRowsPerLoad; ++e) v[e] = list[D::kRowsPerLoad * (wq + NWQ * i) + e];
          at.k[i] = by_lanes(v);
        }
        const uint32_t l = lane_here();
        at.mask = ~0u;
        if (leftP < kBN) {  // past its end the list's last row is repeated
          at.mask = (1u << leftP) - 1u;
          const uint32_t end = list[leftP - 1];
#pragma unroll
          for (int i = 0; i < D::kLoads; ++i)
            if (static_cast<int>(D::kRowsPerLoad * (wq + NWQ * i) + l / kChunks) >= leftP) at.k[i] = end;
        }
#pragma unroll
        for (int i = 0; i < D::kLoads; ++i) at.k[i] += k_chunk(l);
        listP += kBN, leftP -= kBN;
        --tP;  // no tile in rows
      } else {
        const ConstU32 words = words_of(P);
        while (tP < P.tile * (kBM / kBN) && wordP == 0u) wordP = words[++tP];
        at.mask = wordP;
        wordP = words[tP + 1];  // on its way until the next tile (behind the item's last tile a word that no one looks at)
        const int lim = lastP - tP * kBN;
        at.lo = baseP + static_cast<uint64_t>(static_cast<uint32_t>(tP * kBN)) * row_bytes;
#pragma unroll
        for (int i = 0; i < D::kLoads; ++i) at.k[i] = k_lane[i % kHalfLoads] + (first_rows(i) ? 0 : kPage * row_bytes);
        if (__builtin_expect(lim < kBN - 1, 0)) {  // rows past the last key repeat it
          const uint32_t l = lane_here();
#pragma unroll
          for (int i = 0; i < D::kLoads; ++i) {
            const int rr = D::kRowsPerLoad * (wq + NWQ * i) + static_cast<int>(l / kChunks);
            at.k[i] = static_cast<uint32_t>(rr < lim ? rr : lim) * row_bytes + k_chunk(l);
          }
        }
      }
    } else if (paged) {
      at.lim = lastP - tP * kBN;
      at.lo = baseP + static_cast<int64_t>(pg_lo) * (2 * page_half);
      at.hi = baseP + static_cast<int64_t>(pg_hi) * (2 * page_half);
    } else {
      at.lim = lastP - tP * kBN;
      at.lo = baseP + static_cast<uint64_t>(static_cast<uint32_t>(tP * kBN)) * row_bytes;
      at.hi = at.lo + kPage * row_bytes;
    }
    ++tP;
    if (__builtin_expect(tP > lastP / kBN, 0)) {  // the item's last tile: the stream goes on with the block's next item
      const Item it = locate(item_of(jP + 1));
      if (uniform(it.valid)) {
        ++jP;
        P = it;
        enter();
      } else {
        ended = true;
      }
    }
    if (!ended) fetch_page_ids();
    return at;
  };
  auto uniform_ptr = [&](const char* p) DLLAVA_INLINE {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const char*>(static_cast<uint64_t>(static_cast<uint32_t>(uniform(static_cast<int>(v >> 32)))) << 32 |
                                         static_cast<uint32_t>(uniform(static_cast<int>(v))));
  };
  // loads of one half-stage (K or V) of a tile to the LDS address dst
  auto request = [&](const TileAt& at, int64_t step, const uint32_t (&lane_off)[kHalfLoads], bool is_v, uint32_t dst) DLLAVA_INLINE {
    if constexpr (kMasks) {
      const char *lo = at.lo + step, *hi = lo;
      base_ready(lo, hi);
#pragma unroll
      for (int i = 0; i < D::kLoads; ++i) load_to_lds(lo, is_v ? at.k[i] ^ v_flip : at.k[i], dst + (wq + NWQ * i) * (kWave * 16));
      return;
    }
    const char *lo = uniform_ptr(at.lo) + step, *hi = paged ? uniform_ptr(at.hi) + step : lo + kPage * row_bytes;
    uint32_t o[D::kLoads];
#pragma unroll
    for (int i = 0; i < D::kLoads; ++i) o[i] = lane_off[i % kHalfLoads];
    if (__builtin_expect(at.lim < kBN - 1, 0)) {  // rows past the last key repeat it
      const int l = lane_here();
#pragma unroll
      for (int i = 0; i < D::kLoads; ++i) {
        const int rr = D::kRowsPerLoad * (wq + NWQ * i) + l / kChunks, pc = l % kChunks, row = rr < at.lim ? rr : at.lim;
        o[i] = static_cast<uint32_t>(row % kPage) * row_bytes + 16 * (pc ^ (is_v ? 4 * (rr % (kChunks / 4)) : D::k_swizzle(rr)));
      }
      if (at.lim < kPage) hi = lo;
    }
    base_ready(lo, hi);
#pragma unroll
    for (int i = 0; i < D::kLoads; ++i) {
      load_to_lds(first_rows(i) ? lo : hi, o[i], dst + (wq + NWQ * i) * (kWave * 16));
    }
  };
  const uint32_t sK0 = lds_address(sK), sV0 = lds_address(sV);
  constexpr uint32_t kSlot = kTileElems * 2;
  TileAt behind;       // the tile whose K was requested last: its V is next
  uint32_t mask0 = 0, mask1 = 0, mask2 = 0;  // with masks: of the stream's next three tiles
  bool asked = false;  // the latest round requested both (else the stream has ended: there was no K, or neither)
  auto request_v = [&](uint32_t slot) DLLAVA_INLINE {
    if (__builtin_expect(asked, 1)) request(behind, v_step, v_lane, true, sV0 + slot);
  };
  auto request_k = [&](uint32_t slot) DLLAVA_INLINE {
    asked = !ended;
    if constexpr (kMasks) mask0 = mask1, mask1 = mask2;
    if (__builtin_expect(asked, 1)) {
      behind = next_tile_at();
      if constexpr (kMasks) mask2 = behind.mask;
      request(behind, 0, k_lane, false, sK0 + slot);
    }
  };

  // K(0), V(0), K(1), V(1), K(2); iteration t then requests V(t+2) and K(t+3)
  const int tile_first = wave_tile(C, 0);
  request_queries(C, tile_first, 0, kQLoads);
  enter();
  fetch_page_ids();
  request_k(0);
#pragma unroll 1
  for (uint32_t slot = 0; slot < 2 * kSlot; slot += kSlot) {
    request_v(slot);
    request_k(slot + kSlot);
  }
  // the queries and K(0), the oldest of them
  if (asked)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * D::kLoads) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  uint32_t s0 = 0, s1 = kSlot, s2 = 2 * kSlot;  // ring slots of K and V of the tile at hand, the next, the one after
  int tile = tile_first;
  for (;;) {  // items
    // Keys are numbered as they come in the stream: at the item's own rows `skipped` fewer than in the sequence.
    const int skipped = hidden(C) * kBN, nC = C.n - skipped;
    const int lastC = (last_key_of(C) - skipped) / kBN;
    const int last = kFull || tile < 0 ? (tile < 0 ? -1 : lastC) : tile - skipped / kBN;  // this wave's last key tile; -1: it has no queries
    const int q0 = tile * 32;
    int t = 0;
    f32x16 SA, SB;
    Probs P2;
    if (t <= last) {
      // K of C's first tile has landed, and its queries: scores (0)
      const uint32_t kfirst = kb0 + s0, qb = lds_address(myQ) + k_row;
      static_for<kKS>([&](auto I) DLLAVA_INLINE {
        T.q[I.value] = lds_read16_acc<0>(qb ^ (I.value * 32));
        T.k[I.value] = lds_read16_acc<0>(kfirst ^ (I.value * 32));
      });
      lds_wait();
      static_for<kKS>([&](auto I) DLLAVA_INLINE {
        tie4_acc(T.q[I.value]);
        tie4_acc(T.k[I.value]);
      });
      static_for<kKS>([&](auto I) DLLAVA_INLINE {
        if constexpr (I.value == 0) qk_first(SA, T.k[0], T.q[0]); else qk_next(SA, T.k[I.value], T.q[I.value]);
        if constexpr (I.value % (kKS / kNB) == 0) {
          zero_o(T.o[I.value / (kKS / kNB)]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      T.m_ref = kNoReference;
      T.thr = T.m_ref + kSlack;
      T.l_run = 0.f;
    }
    const Item next = locate(item_of(++jC));
    const int next_wave_tile = wave_tile(next, jC);
    int q_next = next.valid ? 0 : kQLoads;  // query loads of the next item issued so far
    bool q_late = false;                    // some of them after the latest wait
    // Every key tile begins alike: V of this tile and K of the next one of the stream must have landed (this wave's loads:
    // the two half-stages requested in the latest iteration may stay in flight; whatever else is in flight -- queries,
    // output stores -- only makes the wait longer; the kernel must not spill registers, scratch traffic would count too: the
    // tests check the build's resource report).  The barrier makes every wave's part visible and says that all waves have
    // read what the requests below overwrite.
    uint32_t kb, vb, kmask = 0;
    auto open = [&]() DLLAVA_INLINE {
      if (__builtin_expect(asked, 1))
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * D::kLoads) : "memory");
      else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      vb = vb0 + s0;
      kb = kb0 + s1;
      if constexpr (kMasks) kmask = mask0;
    };
    auto open_v = [&]() DLLAVA_INLINE {
      q_late = false;
      if (__builtin_expect(q_next < kQLoads, 0)) {
        request_queries(next, next_wave_tile, q_next, q_next + 2);
        q_next += 2;
        q_late = true;
      }
      request_v(s2);
    };
    auto open_k = [&]() DLLAVA_INLINE {
      request_k(s0);
      const uint32_t s3 = s0;
      s0 = s1, s1 = s2, s2 = s3;
    };
    auto any_mask = [&](f32x16& S) DLLAVA_INLINE {
      if constexpr (kMasks) mask_scores(S, t, last, nC, kmask);
    };
    // On entry of the loop: scores of tile t in SB, V and the probabilities of the tile before pending.  (The two score buffers
    // take turns; a loop that can be left in its middle, or entered there, makes the compiler move accumulators.)
    if (t <= last) {
      if ((last - t) & 1) {  // an even number of tiles
        step<DH, true, true>(T, SA, SB, P2, kb, vb, aScale, open, any_mask, open_v, open_k);
        ++t;
      } else {  // an odd number: pairs from the first tile on, behind products with probabilities of zero
        products_done();  // the copy reads the scores
        tie_s(SA);
        SB = SA;
        if constexpr (kMasks) kmask = mask0;
        if (kMasks || t == last) mask_scores(SB, t, last, nC, kmask);
        first_reference(T, SB, aScale);
        P2.hi[0] = P2.hi[1] = P2.lo[0] = P2.lo[1] = u32x4{0u, 0u, 0u, 0u};
        static_for<4 * kNB>([&](auto I) DLLAVA_INLINE { T.v[I.value % kNB][I.value / (2 * kNB)][(I.value / kNB) % 2] = u32x2{0u, 0u}; });
        asm volatile("s_nop 1" ::: "memory");
      }
      while (t < last) {
        step<DH, false, true>(T, SB, SA, P2, kb, vb, aScale, open, any_mask, open_v, open_k);
        ++t;
        step<DH, false, true>(T, SA, SB, P2, kb, vb, aScale, open, any_mask, open_v, open_k);
        ++t;
      }
      step<DH, false, false>(T, SB, SA, P2, kb, vb, aScale, open,
                             [&](f32x16& S) DLLAVA_INLINE { mask_scores(S, t, last, nC, kmask); },  // the diagonal, or the end of the sequence
                             open_v, open_k);
      ++t;
      finish<DH>(T, P2);
    }
    while (t <= lastC) {  // later waves of the block have more tiles
      open();
      open_v();
      open_k();
      ++t;
    }
    if (q_next < kQLoads) {
      request_queries(next, next_wave_tile, q_next, kQLoads);
      q_late = true;
    }
    if (q_late) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // ahead of the stores: those need not be waited for
    if (tile >= 0) store_item(q0, C);
    if (!next.valid) break;
    C = next;
    tile = next_wave_tile;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the stream's end write LDS that must still be this block's
}

// The blocks of a persistent launch: as many as fit the chip at once, found once per kernel.
template <typename Kernel>
int64_t resident_blocks(Kernel kernel, int threads, std::atomic<int64_t>& cached) {
  if (const int64_t known = cached.load(std::memory_order_relaxed)) return known;  // the same value whichever thread gets here first
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0)
    per_cu = 2;
  const int64_t blocks = static_cast<int64_t>(cus) * per_cu;
  cached.store(blocks, std::memory_order_relaxed);
  return blocks;
}

// Launches `kernel` (blocks of nwq waves) over all items; 1 if there are too many of them.
template <typename Kernel>
int launch_items(Kernel kernel, int nwq, std::atomic<int64_t>& cached_blocks, const char* name, const PrefillArgs& a, int64_t rows, hipStream_t st) {
  const int64_t tiles = ceil_div(rows, nwq * 32) + a.B;  // upper bound on sum_b ceil(n_b / (nwq * 32))
  const int64_t items = tiles * a.H;
  if (items > 0x7fffffffLL) return 1;
  // one item per block when the sequences are too many to be numbered in a wave's lanes (see the kernel)
  const bool persistent = a.B <= kWave;
  const int forced = persistent ? launch_override(DLLAVA_LAUNCH_PREFILL_BLOCKS) : 0;  // tests: few blocks, many items each
  const int64_t slots = forced ? forced : (persistent ? resident_blocks(kernel, nwq * kWave, cached_blocks) : items);
  const dim3 grid(static_cast<unsigned>(items < slots ? items : slots));
  hipLaunchKernelGGL(kernel, grid, dim3(nwq * kWave), 0, st, a);
  DLLAVA_CHECK_LAUNCH(name);
  return DLLAVA_OK;
}

}  // namespace

}  // namespace dllava
