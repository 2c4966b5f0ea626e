// Attention of the training form (Eq. 7 of the paper: the keep mask inside the softmax, over the full token set) on the
// matrix cores, bfloat16.
//
// One work item is (sequence, head, 128 consecutive query rows), served by a block of four waves that walks the key
// tiles (32 keys) up to its diagonal.  K and V tiles go from global memory straight into rings of three LDS buffers each
// (asynchronous loads, two tiles ahead of their use, K one tile before V; one block barrier per tile).
//
// The score tile is computed TRANSPOSED, S^T = K Q^T (keys down the rows, queries across the columns) with
// v_mfma_f32_16x16x32_bf16 (which draws less power than the 32x32x16 form, see gemm_ring.h).  In the result layout a lane
// then holds 4 keys of ONE query per 16 x 16 tile, so the online-softmax maximum is a register reduction plus two lane
// exchanges, and the probabilities are already laid out as the B operand of the second product O^T = V^T P^T: they are split
// in place into two bfloat16 operands (16 significant bits) and never leave registers.  The contraction order of that
// second product is chosen to match the order in which S^T leaves the keys in a lane; V stays row-major ([key][dim]) in LDS
// and the matching A fragments (four consecutive keys of one dim per lane) come from the transposing LDS read.
//
// A wave owns 32 queries as two groups of 16 and alternates: while the softmax of one group is computed, the products of
// the other are issued, two or three vector instructions behind each product (written in that order and pinned by
// scheduling barriers):
//     phase 1 of tile t:  softmax(0, t)  beside  P(1, t-1) V,  K Q(1, t)
//     phase 2 of tile t:  softmax(1, t)  beside  P(0, t) V,    K Q(0, t+1)
// Two such waves share a SIMD (of two blocks, so no barrier ties them).  What bounds it: per 32 queries x 32 keys at
// head size 128 the products take 768 clocks of the matrix pipe, the softmax about 130 vector instructions of 4 to 9
// clocks, masking 60 more; a plain instruction that needs the result of the one before waits for it (11 clocks), which is
// what the second wave hides.  One wave of 64 queries per SIMD with the same interleaving was slower (its tile step took
// 2900 clocks, and the requests of the next tile and the barrier, which then nothing hides, 1300 more).
// Measured, 5608 rows of 8 sequences, 32 heads of 128: 285 -> 111 us; 6000 rows of 2: 975 -> 363 us (before: the kernel of
// prefill_mfma.hip with 32x32x16 products and masks, whose registers left one block per compute unit).
#include <type_traits>

#include "gemm_ring.h"
#include "prefill_args.h"

namespace dllava {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // native vector: always promoted to registers

constexpr int kBN = 32;  // keys per tile

// The lane number, behind a statement: what is derived from it is computed where it stands instead of being kept in
// registers across the tile loop.
__device__ __forceinline__ int recomputed(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// One wave-wide load straight into LDS: 16 bytes per lane from base + offset to lds_addr + 16*lane (wave-uniform base and
// lds_addr).  Written as an instruction for its scalar base: the compiler adds the base in every lane.
__device__ __forceinline__ uint32_t lds_address(bf16_t* p) { return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)p)); }
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t offset, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds_addr) : "memory");
}
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
constexpr int kWaves = 4;  // of a block
template <int DH>
struct Dma {
  static constexpr int kChunks = DH / 8;            // 16-byte chunks per row
  static __device__ __forceinline__ int k_swizzle(int rr) { return DH == 128 ? rr % 16 : (rr >> 1) % 8; }
  static constexpr int kRowsPerLoad = kWave / kChunks;
  static constexpr int kLoads = kBN / (kRowsPerLoad * kWaves);  // wave-wide loads per wave per tile, for K and again for V
  static_assert(kLoads >= 1 && kLoads * kRowsPerLoad * kWaves == kBN, "tile does not divide among the waves");

  // A tile of which only rows 0..lim exist (the others repeat row lim): lo / hi = first rows of its two 16-row halves,
  // rows of a half row_bytes apart.
  static __device__ __forceinline__ void partial(uint32_t dst, const char* lo, const char* hi, uint32_t row_bytes, int lim, bool is_v,
                                                 int wq, int lane_kept) {
    const int lane = recomputed(lane_kept);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int slab = wq + kWaves * i;  // which 1 KiB of the tile
      const int rr = kRowsPerLoad * slab + lane / kChunks, pc = lane % kChunks;
      const int row = rr < lim ? rr : lim;
      const char* src = (row < kPage ? lo : hi) + static_cast<uint32_t>(row % kPage) * row_bytes +
                        16 * (pc ^ (is_v ? 4 * (rr % (kChunks / 4)) : k_swizzle(rr)));
      load_to_lds(src, dst + slab * (kWave * 16));
    }
  }
};

// The running maximum is only a reference point of the exponentials: any value within a few powers of two of the
// true maximum serves.  The accumulators are rescaled only when some query's tile maximum exceeds its reference by
// more than this many powers of two (probabilities then stay below 2^kSlack; their bfloat16 split is relative, so
// nothing is lost), which after the first tile of a sequence is rare.
constexpr float kSlack = 8.f;

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
// The products, with the operand files chosen here: scores, probabilities and V in vector registers (at most 128
// of them: the compiler splits the 256 of a wave evenly), outputs, queries and K in accumulation registers (left to
// itself it keeps some of the queries there and copies them in front of every product).  The compiler does not see their hazards: ten instruction slots (nops, or three other products) stand
// between the last product into a register and the first plain instruction that reads it, and two between a plain write
// and a product.
__device__ __forceinline__ void qk_first(f32x4& s, const u32x4& k, const u32x4& q) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(s) : "a"(k), "a"(q));
}
__device__ __forceinline__ void qk_next(f32x4& s, const u32x4& k, const u32x4& q) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(k), "a"(q));
}
__device__ __forceinline__ void pv(f32x4& o, const u32x4& v, const u32x4& p) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(v), "v"(p));
}
__device__ __forceinline__ void products_done() { asm volatile("s_nop 15\n\ts_nop 3" ::: "memory"); }
__device__ __forceinline__ void tie_s(f32x4& s) { asm volatile("" : "+v"(s)); }
__device__ __forceinline__ void tie_o(f32x4& o) { asm volatile("" : "+a"(o)); }

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
// all-lanes maximum / sum over the four 16-lane rows of a wave (lanes l, l^16, l^32, l^48)
__device__ __forceinline__ float rows_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float y = max2(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const uint32_t w = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return max2(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const uint32_t w = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// One group of 16 queries of a wave.
template <int DH>
struct Group {
  f32x4 s[2];          // scores [16-key half]: lane = query lane%16, keys 16*half + 4*(lane/16) + 0..3
  u32x4 hi, lo;        // probabilities as B operand: elements 0..3 = half 0, 4..7 = half 1
  f32x4 o[DH / 16];    // outputs [16-dim block]: dims 16*block + 4*(lane/16) + 0..3
  u32x4 q[DH / 32];    // queries [32-dim step]
  float m_ref, l_run;
};

// V fragments of a tile: [16-dim block], elements as the probabilities'; K fragments: [16-key half][32-dim step]
template <int DH>
struct Frags {
  u32x4 k[2][DH / 32];
  u32x2 v[DH / 16][2];
};

__device__ __forceinline__ u32x4 join(const u32x2& a, const u32x2& b) { return u32x4{a[0], a[1], b[0], b[1]}; }

// The softmax of group G's scores beside the products of group X: P(X) V if PV, then K Q(X) if QK (with X's scores as
// result).  READ_V: the next tile's V fragments are read (from vb) behind the products of K Q; READ_K: the next tile's K
// fragments (from kb) behind those of P V.  SOFTMAX false: the products alone.
template <int DH, bool SOFTMAX, bool PV, bool QK, bool READ_V, bool READ_K>
__device__ __forceinline__ void phase(Group<DH>& G, Group<DH>& X, Frags<DH>& F, uint32_t kb, uint32_t vb, float scale_log2) {
  constexpr int kDB = DH / 16, kKS = DH / 32, kRowBytes = DH * 2;
  constexpr int kNP = PV ? kDB * 2 : 0, kNQ = QK ? kKS * 2 : 0, kNM = kNP + kNQ;
  static_assert(!READ_V || QK, "V is read behind the products of K Q");
  static_assert(!READ_K || PV, "K is read behind the products of P V");
  auto product = [&](auto Mi) DLLAVA_INLINE {
    constexpr int m = decltype(Mi)::value;
    if constexpr (m < kNP) {
      constexpr int db = m / 2;
      const u32x4 va = join(F.v[db][0], F.v[db][1]);
      if constexpr (m % 2 == 0) pv(X.o[db], va, X.hi); else pv(X.o[db], va, X.lo);
      if constexpr (READ_K && m % 2 == 0 && m / 2 < 2 * kKS) {
        constexpr int ks = (m / 2) / 2, half = (m / 2) % 2;
        F.k[half][ks] = lds_read16_acc<half * 16 * kRowBytes>(kb ^ (ks * 64));
      }
    } else {
      constexpr int q = m - kNP, ks = q / 2, half = q % 2;
      if constexpr (READ_K && q == 0) {  // the K fragments requested behind P V
        lds_wait();
        static_for<2 * kKS>([&](auto I) DLLAVA_INLINE { tie4_acc(F.k[I.value % 2][I.value / 2]); });
      }
      if constexpr (ks == 0) qk_first(X.s[half], F.k[half][ks], X.q[ks]);
      else qk_next(X.s[half], F.k[half][ks], X.q[ks]);
      if constexpr (READ_V) {
        constexpr int per = (2 * kDB + kNQ - 1) / kNQ;  // reads behind each product
        static_for<per>([&](auto I) DLLAVA_INLINE {
          constexpr int r = q * per + decltype(I)::value;
          if constexpr (r < 2 * kDB) F.v[r / 2][r % 2] = lds_read8_tr16<(r % 2) * 16 * kRowBytes>(vb ^ ((r / 2) * 32));
        });
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (!SOFTMAX) {
    static_for<kNM>(product);
  } else {
    // the maximum, beside the first products (the fourth one on: the scores' own last product must have been written)
    constexpr int kHead = 6;
    static_assert(kNM > kHead, "the maximum is hidden behind products");
    float tmax;
    static_for<kHead>([&](auto Mi) DLLAVA_INLINE {
      constexpr int m = decltype(Mi)::value;
      product(Mi);
      if constexpr (m == 3) {
        const float x = max3(G.s[0][0], G.s[0][1], G.s[0][2]), y = max3(G.s[0][3], G.s[1][0], G.s[1][1]);
        tmax = max2(max3(x, G.s[1][2], G.s[1][3]), y);
        here(tmax);
      }
      if constexpr (m == 4) {
        tmax = rows_max(tmax);
        here(tmax);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // scale > 0: the maximum of the scaled scores; -inf for a query that sees no key of this tile (possible with key
    // masks only).  m_ref starts at a finite floor, so such a tile leaves the query's state as it is (p = 0).
    const float m_t = tmax * scale_log2;
    if (__any(m_t > G.m_ref + kSlack)) {
      const float m_new = max2(G.m_ref, m_t);
      const float alpha = __builtin_amdgcn_exp2f(G.m_ref - m_new);
      G.m_ref = m_new;
      G.l_run *= alpha;
      static_for<kDB>([&](auto I) DLLAVA_INLINE {
        G.o[I.value] *= alpha;
        tie_o(G.o[I.value]);  // back to accumulation registers here, not in front of the products
      });
    }
    // Probabilities as TWO bfloat16 operands, p = p_hi + p_lo with p_hi the top 16 bits of p and p_lo the top 16 bits of
    // the (exact) remainder: 16 significant bits in all, so the second product is as accurate as the float32
    // accumulation around it.  Four steps of three or four instructions for each of the four pairs.
    float p0, p1, e1, r0;
    auto step = [&](auto Ui) DLLAVA_INLINE {
      constexpr int pr = decltype(Ui)::value / 4, u = decltype(Ui)::value % 4;
      constexpr int half = pr / 2, r = 2 * (pr % 2);
      if constexpr (u == 0) {
        e1 = __builtin_fmaf(G.s[half][r + 1], scale_log2, -G.m_ref);
        p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(G.s[half][r], scale_log2, -G.m_ref));
      } else if constexpr (u == 1) {
        p1 = __builtin_amdgcn_exp2f(e1);
        r0 = p0 - __uint_as_float(__float_as_uint(p0) & 0xffff0000u);
      } else if constexpr (u == 2) {
        uint32_t h = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u);  // {hi16(p0), hi16(p1)}
        here(h);
        G.hi[pr] = h;
        G.l_run += p0;
        G.l_run += p1;
        here(G.l_run);
      } else {
        const float r1 = p1 - __uint_as_float(__float_as_uint(p1) & 0xffff0000u);
        uint32_t l = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
        here(l);
        G.lo[pr] = l;
      }
    };
    constexpr int kRest = kNM - kHead;
    static_for<kRest>([&](auto Ri) DLLAVA_INLINE {
      constexpr int i = decltype(Ri)::value, u0 = i * 16 / kRest, u1 = (i + 1) * 16 / kRest;
      product(std::integral_constant<int, kHead + i>{});
      static_for<u1 - u0>([&](auto U) DLLAVA_INLINE { step(std::integral_constant<int, u0 + decltype(U)::value>{}); });
      __builtin_amdgcn_sched_barrier(0);
    });
  }
}

// One work item = (sequence, head, tile of 128 query rows).  Blocks are PERSISTENT: the launch holds as many blocks as
// fit the chip at once (slots), block p takes every slots-th item and walks their key tiles as ONE stream: the tile
// loads run two tiles ahead of the arithmetic across item boundaries, and the queries of the next item go to LDS while
// the current item runs.  A block that starts needs three or four dependent trips to memory before its first tile; a
// persistent block pays them once.
// Items are numbered by DESCENDING query-tile index over all sequences, heads adjacent: a causal item's work grows
// with its tile index, so every block takes its longest items first and the launch ends with the shortest ones.
template <int DH>
__global__ __launch_bounds__(kWaves * kWave, 2) void masked_mfma_kernel(PrefillArgs args, int items_cap) {
  // the arguments as locals (the closures below then capture plain values, which the compiler keeps in registers)
  const int aB = args.B;
  const float aScale = args.scale_log2;
  const void* const aK = args.K;
  const void* const aV = args.V;
  void* const aO = args.O;
  constexpr int kBM = kWaves * 32;
  constexpr int kChunks = DH / 8;  // 16-byte chunks per row
  constexpr int kDB = DH / 16;     // 16-dim blocks of the output
  constexpr int kKS = DH / 32;     // 32-dim steps of the first product
  constexpr int kRowBytes = DH * 2;
  constexpr int kTileElems = kBN * DH;
  constexpr int kStages = 3;
  using D = Dma<DH>;

  // rings of three K tiles and three V tiles, and every wave's 32 queries of the block's next item (together half of a
  // compute unit's LDS at most: two blocks share it)
  __shared__ __align__(1024) bf16_t sK[kStages * kTileElems];
  __shared__ __align__(1024) bf16_t sV[kStages * kTileElems];
  __shared__ __align__(1024) bf16_t sQ[kWaves * 32 * DH];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wq = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int H = args.H;
  const int g = lane >> 4, lq = lane & 15;
  // Offsets and mask words were written by earlier launches and do not change while this kernel runs:
  // read through the constant address space, block-uniform indices become scalar loads.  (As plain pointers they
  // may alias the output, which this kernel now stores inside its loop, and every one of them would be a vector
  // load with a full vector-memory wait behind it -- a wait for the tile loads in flight.)
  typedef const int32_t __attribute__((address_space(4)))* ConstI32;
  typedef const uint32_t __attribute__((address_space(4)))* ConstU32;
  const ConstI32 off_c = (ConstI32)args.off;
  const ConstU32 kw_c = (ConstU32)args.key_words;
  const int step = static_cast<int>(gridDim.x);

  // Which (sequence, query tile) is item k?  With at most 64 sequences every wave keeps the sequences' offsets in
  // its lanes (lane = sequence; one trip to memory per block) and counts with ballots; with more, the sequences are
  // walked with scalar loads (then there is one item per block).
  const bool by_lane = aB <= kWave;
  int off_l = 0, end_l = 0, nb_l = 0, total = 0;
  if (by_lane) {
    off_l = lane < aB ? off_c[lane] : 0;
    end_l = lane < aB ? off_c[lane + 1] : 0;
    // The offsets have arrived; the statement also tells the compiler so: it would otherwise order every later use
    // of them, in loops it cannot see through, behind ALL outstanding vector-memory operations -- the tile loads.
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(off_l), "+v"(end_l));
    nb_l = (end_l - off_l + kBM - 1) / kBM;  // tiles of sequence `lane`
    int cnt = 0;
    for (int i = 0; (cnt = __builtin_popcountll(__ballot(nb_l > i))) != 0; ++i) total += cnt;
  }
  struct Item {
    int valid, b, h, tile, r0, n;
  };
  // Many sequences, one item per block: numbered sequence by sequence, the late (long) tiles of each first.  Found once, 64
  // sequences at a time (as a scalar walk, a chain of loads, 500 sequences of one row and 8 heads took 199 us, now 45).
  Item only{0, 0, 0, 0, 0, 0};
  if (!by_lane) {
    int tile = static_cast<int>(blockIdx.x) / H;
    for (int b0 = 0; b0 < aB; b0 += kWave) {
      const int b = b0 + lane;
      const int r0 = b < aB ? off_c[b] : 0, n = b < aB ? off_c[b + 1] - r0 : 0;
      const int nt = (n + kBM - 1) / kBM, upto = wave_incl_scan(nt);  // tiles of the sequences up to this lane's
      const unsigned long long past = __ballot(upto > tile);
      if (past) {
        const int l = __builtin_ctzll(past);
        // the sequence's first tile is number upto - nt, its last upto - 1: counted from the last
        only = {1, b0 + l, 0, __builtin_amdgcn_readlane(upto, l) - 1 - tile, __builtin_amdgcn_readlane(r0, l), __builtin_amdgcn_readlane(n, l)};
        break;
      }
      tile -= __builtin_amdgcn_readlane(upto, kWave - 1);
    }
  }
  auto locate = [&](int k) __attribute__((always_inline)) {
    Item it{0, 0, 0, 0, 0, 0};
    if (k >= items_cap) return it;
    const int yd = k / H;  // position in DESCENDING tile-index order
    it.h = k - yd * H;
    if (by_lane) {
      const int y = total - 1 - yd;  // position in ascending order
      if (y < 0) return it;
      int below = 0, tile = 0;  // tiles with a smaller index
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
      it.b = __builtin_ctzll(me);
      it.tile = tile;
      it.r0 = __builtin_amdgcn_readlane(off_l, it.b);
      it.n = __builtin_amdgcn_readlane(end_l, it.b) - it.r0;
      it.valid = 1;
    } else {
      if (k == static_cast<int>(blockIdx.x)) it = only, it.h = k - yd * H;
    }
    return it;
  };
  // keys 0..last_key of its sequence are needed by an item
  auto last_key_of = [&](const Item& it) __attribute__((always_inline)) { return (it.tile * kBM + kBM < it.n ? it.tile * kBM + kBM : it.n) - 1; };

  // Round j of block p takes item p + j*step, in odd rounds (step-1-p) + j*step: the rounds run through the items
  // (sorted by descending work) in alternating directions, so a block that got a longer item in one round gets a
  // shorter one in the next and the blocks' totals stay close (C5 shape: 40..42 tiles per block instead of 36..46).
  const int pblk = static_cast<int>(blockIdx.x);
  auto item_of = [&](int j) __attribute__((always_inline)) { return ((j & 1) ? step - 1 - pblk : pblk) + j * step; };
  int jC = 0;
  Item C = locate(item_of(0));
  if (!C.valid) return;

  // ---- the two query groups of this wave: 16 queries each of its 32-query tile --------------------------------------------
  Group<DH> G0, G1;
  // Which 32-query tile of an item: in every other item of a block the waves take them the other way round, so the SIMDs
  // share the longer causal tiles.  -1: none.
  auto wave_tile = [&](const Item& it, int j) DLLAVA_INLINE {
    const int t = it.tile * kWaves + ((j ^ (pblk >> 8)) & 1 ? kWaves - 1 - wq : wq);
    return it.valid && t * 32 < it.n ? t : -1;
  };
  const bf16_t* Qp = static_cast<const bf16_t*>(args.Q);
  constexpr int kQLoads = 32 / D::kRowsPerLoad;  // wave-wide loads of a wave's 32 query rows
  bf16_t* myQ = sQ + wq * 32 * DH;
  auto request_queries = [&](const Item& it, int tile, int from, int to) DLLAVA_INLINE {  // loads from .. to-1 of a wave's queries
    const int l = recomputed(lane);
    for (int i = from; i < to; ++i) {
      const int rr = D::kRowsPerLoad * i + l / kChunks, pc = l % kChunks;
      int q = (tile < 0 ? 0 : tile * 32) + rr;
      if (q >= it.n) q = it.n - 1;
      const bf16_t* src = Qp + (static_cast<size_t>(it.r0 + q) * H + it.h) * DH + 8 * (pc ^ D::k_swizzle(rr));
      load_to_lds(reinterpret_cast<const char*>(src), lds_address(myQ) + i * (kWave * 16));
    }
  };
  auto mask_word = [&](const Item& it, int t) DLLAVA_INLINE { return kw_c[(it.r0 >> 5) + it.b + t]; };
  // The key tiles of an item, in order.  Tiles whose keys are all hidden and hold none of the item's own
  // queries are left out of the stream.
  auto shown = [&](const Item& it, int t) DLLAVA_INLINE {
    while (t * kBN + kBN - 1 < it.tile * kBM && mask_word(it, t) == 0u) ++t;
    return t;
  };

  // Fragment addresses (LDS bytes, stage 0).  K: row lq (+16), logical chunk 4*ks + g, stored at chunk ^ swizzle(lq): the
  // step ks enters as an exclusive-or with 64*ks.  Queries alike.  V: the transposing read of 16 lanes (j = lane mod 16)
  // returns to lane j four keys of dim j; lane j points at key 4*g + j/4, dims 4*(j mod 4)..+3 of a 16-dim block; the
  // block enters as an exclusive-or with 32*block.
  const uint32_t k_row = lq * kRowBytes + ((g ^ D::k_swizzle(lq)) * 16);
  const uint32_t kb0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)sK)) + k_row;
  const uint32_t qb0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)myQ)) + k_row;
  const uint32_t vb0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DLLAVA_LDS bf16_t*)sV)) +
                       (4 * g + (lq >> 2)) * kRowBytes + ((lq >> 2) % (kChunks / 4)) * 64 + (lq & 3) * 8;

  auto begin_group = [&](Group<DH>& G, auto WHICH) DLLAVA_INLINE {
    constexpr int row0 = decltype(WHICH)::value * 16;
    static_for<kKS>([&](auto I) DLLAVA_INLINE { G.q[I.value] = lds_read16_acc<row0 * kRowBytes>(qb0 ^ (I.value * 64)); });
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
      G.o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
      tie_o(G.o[db]);
    }
    G.hi = G.lo = u32x4{0u, 0u, 0u, 0u};
    G.m_ref = -1e30f;  // finite floor, not -inf: see phase()
    G.l_run = 0.f;
  };
  // scores above the diagonal of some query (keys > qi), or hidden by a zero bit of kmask (except the query's own key);
  // q0: first query of the group
  auto mask_scores = [&](Group<DH>& G, int q0, const Item& it, int t, uint32_t kmask) DLLAVA_INLINE {
    const int j0 = t * kBN;
    if (j0 + kBN - 1 > q0 || kmask != ~0u) {
      products_done();
      tie_s(G.s[0]);
      tie_s(G.s[1]);
      const int l = recomputed(lane), g4 = 4 * (l >> 4);
      int qi = q0 + (l & 15);
      if (qi >= it.n) qi = it.n - 1;
      const int self = qi - j0 - g4;  // the query's own key, as kk
      const uint32_t km = kmask >> g4;
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int kk = 16 * half + r;  // key j0 + g4 + kk
          const bool open = (km >> kk) & 1u;
          if (kk > self || (!open && kk != self)) G.s[half][r] = -INFINITY;
        }
    }
  };
  auto store_group = [&](Group<DH>& G, int q0, const Item& it) DLLAVA_INLINE {
    const float inv = 1.f / rows_sum(G.l_run);
    const int l = recomputed(lane), g = l >> 4, qi = q0 + (l & 15);
    bf16_t* orow = static_cast<bf16_t*>(aO) + (static_cast<size_t>(it.r0 + qi) * H + it.h) * DH;
#pragma unroll
    for (int db = 0; db < kDB; db += 2) {
      // a lane holds dims 4*g..+3 of two 16-dim blocks; exchanged with the neighbouring 16 lanes it holds eight
      // consecutive dims of one of them
      const auto a = __builtin_amdgcn_permlane16_swap(pack_bf16x2(G.o[db][0] * inv, G.o[db][1] * inv),
                                                      pack_bf16x2(G.o[db + 1][0] * inv, G.o[db + 1][1] * inv), false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(pack_bf16x2(G.o[db][2] * inv, G.o[db][3] * inv),
                                                      pack_bf16x2(G.o[db + 1][2] * inv, G.o[db + 1][3] * inv), false, false);
      const uint4 piece = {a[0], b[0], a[1], b[1]};
      if (qi < it.n) *reinterpret_cast<uint4*>(orow + 16 * (db + (g & 1)) + 8 * (g >> 1)) = piece;
    }
  };

  // ---- the stream of tile loads: item P, its tile tP is the next one whose K is requested; V follows one tile behind --------
  // A tile is two halves of 16 rows; all of a half's rows lie at fixed offsets from its first, so a tile's loads are a
  // scalar base plus a lane constant each.
  const uint32_t row_bytes = static_cast<uint32_t>(H) * kRowBytes;
  const int64_t v_step = static_cast<const char*>(aV) - static_cast<const char*>(aK);
  constexpr int kHalfLoads = D::kLoads >= 2 ? D::kLoads / 2 : 1;  // distinct row sets of a wave within a half
  uint32_t k_lane[kHalfLoads], v_lane[kHalfLoads];
#pragma unroll
  for (int i = 0; i < kHalfLoads; ++i) {
    const int rr = D::kRowsPerLoad * (wq + kWaves * i) + lane / kChunks, pc = lane % kChunks;
    k_lane[i] = (rr % kPage) * row_bytes + 16 * (pc ^ D::k_swizzle(rr));
    v_lane[i] = (rr % kPage) * row_bytes + 16 * (pc ^ (4 * (rr % (kChunks / 4))));
  }
  struct TileAt {
    const char* at;  // K of the tile's first row, this head
    int lim;         // last row of the tile that exists (>= kBN - 1: all of them)
  };
  int jP = 0, tP, lastP;
  const char* baseP;  // K of the first row of P's sequence, its head
  Item P = C;
  auto uniform = [](int v) DLLAVA_INLINE { return __builtin_amdgcn_readfirstlane(v); };  // said to the compiler where it cannot see it
  auto enter = [&]() DLLAVA_INLINE {  // the stream enters item P
    P.b = uniform(P.b), P.h = uniform(P.h), P.tile = uniform(P.tile), P.r0 = uniform(P.r0), P.n = uniform(P.n);
    lastP = last_key_of(P);
    baseP = static_cast<const char*>(aK) + static_cast<int64_t>(P.r0) * row_bytes + P.h * kRowBytes;
    tP = uniform(shown(P, 0));
  };
  auto next_tile_at = [&]() DLLAVA_INLINE {  // tile tP of item P; then on to the next tile of the stream
    const TileAt at{baseP + static_cast<uint64_t>(static_cast<uint32_t>(tP * kBN)) * row_bytes, lastP - tP * kBN};
    const int t_before = tP;
    tP = shown(P, tP + 1);
    if (__builtin_expect(tP > lastP / kBN, 0)) {  // the item's last tile: the stream goes on with the block's next item
      const Item it = locate(item_of(jP + 1));
      if (uniform(it.valid)) {
        ++jP;
        P = it;
        enter();
      } else {
        tP = t_before;  // the stream has ended: its last tile once more (never used; no case of its own for every tile)
      }
    }
    return at;
  };
  // loads of one half-stage (K or V) of a tile to the LDS address dst
  auto request = [&](const TileAt& tile_at, int64_t step, const uint32_t (&lane_off)[kHalfLoads], bool is_v, uint32_t dst) DLLAVA_INLINE {
    const char *lo = tile_at.at + step, *hi = lo + kPage * row_bytes;
    if (__builtin_expect(tile_at.lim >= kBN - 1, 1)) {
#pragma unroll
      for (int i = 0; i < D::kLoads; ++i) {
        const int slab = wq + kWaves * i;
        load_to_lds(D::kRowsPerLoad * slab < kPage ? lo : hi, lane_off[i % kHalfLoads], dst + slab * (kWave * 16));
      }
    } else {  // rows past the last key repeat it (see Dma)
      D::partial(dst, lo, hi, row_bytes, tile_at.lim, is_v, wq, lane);
    }
  };
  const uint32_t sK0 = lds_address(sK), sV0 = lds_address(sV);
  constexpr uint32_t kSlot = kTileElems * 2;
  TileAt behind;  // the tile whose K was requested last: its V is next
  auto request_k = [&](uint32_t slot) DLLAVA_INLINE {
    behind = next_tile_at();
    request(behind, 0, k_lane, false, sK0 + slot);
  };
  auto request_v = [&](uint32_t slot) DLLAVA_INLINE { request(behind, v_step, v_lane, true, sV0 + slot); };

  // K(0), V(0), K(1), V(1), K(2); iteration t then requests V(t+2) and K(t+3)
  const int tile_first = wave_tile(C, 0);
  request_queries(C, tile_first, 0, kQLoads);
  enter();
  request_k(0);
  request_v(0);
  request_k(kSlot);
  request_v(kSlot);
  request_k(2 * kSlot);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * D::kLoads) : "memory");  // the queries and K(0), the oldest of them
  __builtin_amdgcn_s_barrier();

  Frags<DH> F;
  uint32_t s0 = 0, s1 = kSlot, s2 = 2 * kSlot;  // ring slots of K and V of the tile at hand, the next, the one after
  int tile = tile_first;
  for (;;) {  // items
    const int lastC = last_key_of(C) / kBN;
    const int last = tile;  // this wave's last key tile; -1: it has no queries
    const int q0 = tile * 32;
    // K of C's first tile has landed, and its queries
    int t = shown(C, 0);
    begin_group(G0, std::integral_constant<int, 0>{});
    begin_group(G1, std::integral_constant<int, 1>{});
    const uint32_t kfirst = kb0 + s0;
    static_for<2 * kKS>([&](auto I) DLLAVA_INLINE {
      constexpr int half = decltype(I)::value % 2, ks = decltype(I)::value / 2;
      F.k[half][ks] = lds_read16_acc<half * 16 * kRowBytes>(kfirst ^ (ks * 64));
    });
#pragma unroll
    for (int db = 0; db < kDB; ++db) F.v[db][0] = F.v[db][1] = u32x2{0u, 0u};
    lds_wait();
    static_for<2 * kKS>([&](auto I) DLLAVA_INLINE { tie4_acc(F.k[I.value % 2][I.value / 2]); });
    static_for<kKS>([&](auto I) DLLAVA_INLINE {
      tie4_acc(G0.q[I.value]);
      tie4_acc(G1.q[I.value]);
    });
    asm volatile("s_nop 7" ::: "memory");  // plain writes of the accumulators before the first product
    phase<DH, false, false, true, false, false>(G0, G0, F, 0, 0, aScale);
    const Item next = locate(item_of(++jC));
    const int next_wave_tile = wave_tile(next, jC);
    int q_next = next.valid ? 0 : kQLoads;  // query loads of the next item issued so far
    bool q_late = false;                    // some of them after the latest wait
    // Every key tile begins alike: V of this tile and K of the next one of the stream must have landed (this wave's loads:
    // the two half-stages requested in the latest iteration may stay in flight; whatever else is in flight -- queries,
    // output stores -- only makes the wait longer; the kernel must not spill registers, scratch traffic would count too: the
    // tests check the build's resource report).  The barrier makes every wave's part visible and says that all waves have
    // read what the requests below overwrite.  (What stands here is paid by both waves of a SIMD for every tile: scalar
    // arithmetic in dependent steps and branches took 1100 clocks before it was cut to what it is.)
    uint32_t kb, vb, kmask;
    auto open_tile = [&]() DLLAVA_INLINE {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * D::kLoads) : "memory");
      __builtin_amdgcn_s_barrier();
      q_late = false;
      if (__builtin_expect(q_next < kQLoads, 0)) {
        request_queries(next, next_wave_tile, q_next, q_next + 2);
        q_next += 2;
        q_late = true;
      }
      request_v(s2);
      request_k(s0);
      vb = vb0 + s0;
      kb = kb0 + s1;
      const uint32_t s3 = s0;
      s0 = s1, s1 = s2, s2 = s3;
      kmask = mask_word(C, t);
    };
    // On entry of a tile K(t) is in F.k, V of the tile before and P(1) of it are pending, scores (0, t) are computed.
    while (t <= last) {
      open_tile();
      mask_scores(G0, q0, C, t, kmask);
      phase<DH, true, true, true, true, false>(G0, G1, F, kb, vb, aScale);   // softmax(0,t) | P(1) V, K Q(1,t), V(t) read
      lds_wait();
      static_for<2 * kDB>([&](auto I) DLLAVA_INLINE { tie2(F.v[I.value / 2][I.value % 2]); });
      mask_scores(G1, q0 + 16, C, t, kmask);
      phase<DH, true, true, true, false, true>(G1, G0, F, kb, vb, aScale);   // softmax(1,t) | P(0) V, K(t+1) read, K Q(0,t+1)
      t = shown(C, t + 1);
    }
    while (t <= lastC) {  // later waves of the block have more tiles
      open_tile();
      t = shown(C, t + 1);
    }
    if (q_next < kQLoads) {
      request_queries(next, next_wave_tile, q_next, kQLoads);
      q_late = true;
    }
    // the last P(1) V of the item, then its outputs
    if (tile >= 0) {
      phase<DH, false, true, false, false, false>(G1, G1, F, 0, 0, aScale);
      products_done();
      static_for<kDB>([&](auto I) DLLAVA_INLINE {
        tie_o(G0.o[I.value]);
        tie_o(G1.o[I.value]);
      });
    }
    if (q_late) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // ahead of the stores: those need not be waited for
    if (tile >= 0) {
      store_group(G0, q0, C);
      store_group(G1, q0 + 16, C);
    }
    if (!next.valid) break;
    C = next;
    tile = next_wave_tile;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the stream's end write LDS that must still be this block's
}

// blocks that fit the chip at once (persistent launch): compute units x blocks per compute unit, found once per kernel
template <int DH>
int64_t resident_blocks() {
  static int64_t cached = 0;  // the same value whichever thread gets here first
  if (cached) return cached;
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, masked_mfma_kernel<DH>, kWaves * kWave, 0) != hipSuccess || per_cu <= 0)
    per_cu = 2;
  cached = static_cast<int64_t>(cus) * per_cu;
  return cached;
}

// Items of 128 rows whatever the size of the launch: of 480 calls (1 to 64 heads of 64 and 128, 1 to 300 sequences of 8 to 3000
// rows) none is slower than on the 32-, 64- and 128-row items of the kernel before, the closest being one sequence of 1500
// rows, 1 head of 64: 52.6 / 53.5 us; 214 rows, 8 heads of 64: 14.6 / 16.3.
template <int DH>
int launch(const PrefillArgs& a, int64_t rows, hipStream_t st) {
  const int64_t tiles = ceil_div(rows, kWaves * 32) + a.B;  // upper bound on sum_b ceil(n_b / 128)
  const int64_t items = tiles * a.H;
  if (items > 0x7fffffffLL) return 1;
  // one item per block when the sequences are too many to be numbered in a wave's lanes (see the kernel)
  const bool persistent = a.B <= kWave;
  const int forced = persistent ? launch_override(DLLAVA_LAUNCH_PREFILL_BLOCKS) : 0;  // tests: few blocks, many items each
  const int64_t slots = forced ? forced : (persistent ? resident_blocks<DH>() : items);
  const dim3 grid(static_cast<unsigned>(items < slots ? items : slots));
  hipLaunchKernelGGL(masked_mfma_kernel<DH>, grid, dim3(kWaves * kWave), 0, st, a, static_cast<int>(items));
  DLLAVA_CHECK_LAUNCH("masked_mfma_kernel");
  return DLLAVA_OK;
}

}  // namespace

// returns 1 if the shape is not handled here
int masked_mfma_launch(const PrefillArgs& a, int64_t rows, int Dh, hipStream_t st) {
  if (Dh == 128) return launch<128>(a, rows, st);
  if (Dh == 64) return launch<64>(a, rows, st);
  return 1;
}

}  // namespace dllava
