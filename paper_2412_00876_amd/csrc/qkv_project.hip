// dllava_qkv_project: Q, K, V of the REDUCED token set (Eq. 3 line 1 of the paper applied to S^{P*}): the
// projections of the decoder layer run over the kept rows only, which is where the paper's prefill saving comes
// from (Sec. 3.2: most of the cost is in the linear layers; Eq. 13: the 32 B N C^2 term).  Queries and keys are
// rotated by the ORIGINAL position of each kept token (rotary embedding of the LLaMA decoder; the paper does not
// mention positions), queries go to a compacted [rows, H, Dh] tensor, keys and values straight into the paged
// cache, so that compaction has to move hidden states only.
//
//  * qkv_ring_kernel (bfloat16, Dh = 128): the transposed product W . x^T of gemm_ring.h, one block per compute unit: one or
//    two heads of Q, K or V against 64 .. 256 compacted rows.  A wave holds both members of every rotary pair (i, i + 64)
//    it works on, so the rotation happens in registers; the tile is then transposed through LDS (chunk-swizzled) so that
//    every (token, head) row leaves as 256 contiguous bytes.
//  * qkv_generic_kernel: any dtype / head size, one thread per rotary pair of one row.
#include "dllava.h"
#include "gemm_ring.h"

namespace dllava {

int check_cache(const dllava_kv_cache* c, const char* who);

namespace {

struct QkvArgs {
  const void* x;
  int64_t ldx, d;
  int32_t B;
  const int32_t* off;
  const int32_t* pos;  // nullptr: no rotation
  const void* W[3];
  int32_t H, Dh;
  void* Q_out;
  void* pages;
  const int32_t* block_table;
  int32_t* cache_len;
  int32_t max_pages;
  int32_t* err_flag;
};

// rotary angle per position of pair i, in revolutions, as float hi + lo (matrix-core kernel) and as a double in
// radians (generic kernel)
struct RopeTable {
  float hi[64], lo[64];
};
struct RopeTableD {
  double f[64];
};

// sequence of compacted row r: largest b with off[b] <= r
__device__ __forceinline__ int seq_of_row(const int32_t* off, int B, int r) {
  int lo = 0, hi = B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= r) lo = mid; else hi = mid;
  }
  return lo;
}

// element offset of (token j of sequence b, head) inside the pages, K block; the V block is H*kPage*Dh further.
// -1 when j is beyond the capacity of the sequence.
__device__ __forceinline__ int64_t page_slot(const QkvArgs& a, int b, int j, int head) {
  if (j >= a.max_pages * kPage) return -1;
  const int pg = a.block_table[static_cast<size_t>(b) * a.max_pages + j / kPage];
  return ((static_cast<int64_t>(pg) * 2 * a.H + head) * kPage + j % kPage) * a.Dh;
}

// cache_len[b] = min(n_b, capacity); the flag reports an overflow
__device__ __forceinline__ void set_lengths(const QkvArgs& a, int tid, int nthreads) {
  const int cap = a.max_pages * kPage;
  for (int b = tid; b < a.B; b += nthreads) {
    const int n = a.off[b + 1] - a.off[b];
    a.cache_len[b] = n < cap ? n : cap;
    if (n > cap && a.err_flag) *a.err_flag = 1;
  }
}

// FI = 8: feature tile f of matrix `which` = heads 2f and 2f+1 (the second may not exist when H is odd: its weight rows are
// clamped and nothing of it is stored), wave w holds head w/2 of the tile.  FI = 4: one head, wave w holds features
// 32*(w/2) + [0, 32) and 64 + 32*(w/2) + [0, 32): the tile's rows are loaded in that order.
template <int FI, int JB>
__global__ __launch_bounds__(kRingThreads, 1) void qkv_ring_kernel(QkvArgs a, RopeTable rt, int n_ft) {
  constexpr int kTok = 32 * JB, kHeads = FI / 4;
  constexpr int kDepth = kRingLdsBytes / ((FI + JB) * 32 * kRingRowBytes);  // FI < 8: stages that LDS holds
  using Off = std::conditional_t<FI == 8, uint32_t, int64_t>;
  __shared__ __align__(1024) char smem_raw[kRingLdsBytes];
  DLLAVA_LDS char* smem = (DLLAVA_LDS char*)smem_raw;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int total = a.off[a.B];
  const int H = a.H;
  if (blockIdx.x == 0) set_lengths(a, tid, kRingThreads);
  // The tiles that exist are dealt to the dies, not those of the launch, which is sized for the upper bound `rows`: with
  // rows = 4 * off[B] three quarters of the dies would have had nothing (1500 rows of 32 heads, d = 4096: 373 us, now 141).
  const int n_tt = (total + kTok - 1) / kTok, per_xcd = (n_ft * n_tt + kRingXcds - 1) / kRingXcds;
  int ft, tt;  // feature tile (kHeads heads), token tile (kTok compacted rows)
  if (!ring_tile(n_ft, n_tt, per_xcd, ft, tt)) return;
  const int tiles_per_matrix = (H + kHeads - 1) / kHeads;
  const int which = ft / tiles_per_matrix, head0 = kHeads * (ft % tiles_per_matrix);
  const int64_t d = a.d;

  Off ga[FI], gb[JB];
#pragma unroll
  for (int j = 0; j < FI; ++j) {
    const int row = ring_load_row(w, j, lane);
    int64_t f = static_cast<int64_t>(head0) * 128 + (FI == 8 ? row : 32 * (row >> 6) + (row & 31) + 64 * ((row >> 5) & 1));
    if (f >= static_cast<int64_t>(H) * 128) f = static_cast<int64_t>(H) * 128 - 1;
    ga[j] = static_cast<Off>(f * d * 2) + ring_load_chunk_bytes(row, lane);
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int row = ring_load_row(w, j, lane);
    int r = tt * kTok + row;
    if (r >= total) r = total - 1;  // such rows are computed and dropped
    gb[j] = static_cast<Off>(static_cast<int64_t>(r) * a.ldx * 2) + ring_load_chunk_bytes(row, lane);
  }
  ring_f32x4 acc[FI][JB];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) acc[i][j] = ring_f32x4{0.f, 0.f, 0.f, 0.f};
  const char *Ab = static_cast<const char*>(a.W[which]), *Bb = static_cast<const char*>(a.x);
  if constexpr (FI == 8)
    gemm_ring_halves<FI, JB>(Ab, ga, Bb, gb, static_cast<int>(d / kRingBK), smem, w, acc);
  else
    gemm_ring_small<FI, JB, kDepth>(Ab, ga, Bb, gb, static_cast<int>(d / kRingBK), smem, w, acc);
  __syncthreads();  // the ring memory becomes the transposed output tile

  // where the rows of this tile go: one entry per (head of the tile, token)
  bf16_t* sO = reinterpret_cast<bf16_t*>(smem_raw);  // [kTok tokens][16*kHeads chunks of 8 features], chunk c of token t at c ^ (t % 16)
  int64_t* sm_dst = reinterpret_cast<int64_t*>(smem_raw + kTok * 256 * kHeads);  // [kHeads][kTok]
  for (int e = tid; e < kHeads * kTok; e += kRingThreads) {
    const int h2 = e / kTok, t = e % kTok;
    const int r = tt * kTok + t, head = head0 + h2;
    int64_t dst = -1;
    if (r < total && head < H) {
      if (which == 0) {
        dst = (static_cast<int64_t>(r) * H + head) * 128;
      } else {
        const int b = seq_of_row(a.off, a.B, r);
        dst = page_slot(a, b, r - a.off[b], head);
        if (dst >= 0 && which == 2) dst += static_cast<int64_t>(H) * kPage * 128;
      }
    }
    sm_dst[e] = dst;
  }

  // lane: token 16*JB*(w%2) + 16*j + lane%16; register r of acc[i], i < FI/2: feature f_wave + 16*i + 4*(lane/16) + r of the
  // wave's head; acc[i + FI/2] holds the other members of the rotary pairs, 64 features on
  constexpr int kHalf = FI / 2;
  const int f_wave = FI == 8 ? 0 : 32 * (w >> 1);
  const int g = lane >> 4;
  const bool rotate = which < 2 && a.pos;  // block-uniform
  // all of the epilogue's loads at once: the positions of the lane's rows and the revolutions per position of its pairs
  float pos[JB], fh[4 * kHalf], fl[4 * kHalf];
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    int r = tt * kTok + 16 * JB * (w & 1) + 16 * j + (lane & 15);
    if (r >= total) r = total - 1;
    pos[j] = rotate ? static_cast<float>(a.pos[r]) : 0.f;
  }
#pragma unroll
  for (int i = 0; i < kHalf; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      fh[4 * i + r] = rt.hi[f_wave + 16 * i + 4 * g + r];
      fl[4 * i + r] = rt.lo[f_wave + 16 * i + 4 * g + r];
    }
  auto column = [&](auto ROTATE, auto J) DLLAVA_INLINE {
    constexpr int j = decltype(J)::value;
    const int t = 16 * JB * (w & 1) + 16 * j + (lane & 15);
    float v[FI][4];
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      ring_tie_acc(acc[i][j]);  // in accumulation registers until its column: the others do not hold them all
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = acc[i][j][e];
    }
    if constexpr (decltype(ROTATE)::value) {
      const float p = pos[j];
#pragma unroll
      for (int i = 0; i < kHalf; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float hi = fh[4 * i + e];
          const float ph = p * hi;
          const float fr = __builtin_amdgcn_fractf(ph) + (__builtin_fmaf(p, hi, -ph) + p * fl[4 * i + e]);
          const float sn = __builtin_amdgcn_sinf(fr), cs = __builtin_amdgcn_cosf(fr);
          const float x0 = v[i][e], x1 = v[i + kHalf][e];
          v[i][e] = x0 * cs - x1 * sn;
          v[i + kHalf][e] = x1 * cs + x0 * sn;
        }
    }
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      // chunk of 8 features; this lane's half of it: g % 2
      const int c = (FI == 8 ? 16 * (w >> 1) + 2 * i : f_wave / 8 + 2 * (i % kHalf) + 8 * (i / kHalf)) + (g >> 1);
      uint2 o;
      o.x = pack_bf16x2(v[i][0], v[i][1]);
      o.y = pack_bf16x2(v[i][2], v[i][3]);
      *reinterpret_cast<uint2*>(sO + t * (128 * kHeads) + ((c ^ (t & 15)) * 8) + (g & 1) * 4) = o;
    }
    __builtin_amdgcn_sched_barrier(0);  // one column at a time: the accumulators leave no registers for more
  };
  // two copies rather than a branch per column: joining the branches' values costs registers the kernel does not have
  if (rotate)
    static_for<JB>([&](auto J) DLLAVA_INLINE { column(std::true_type{}, J); });
  else
    static_for<JB>([&](auto J) DLLAVA_INLINE { column(std::false_type{}, J); });
  __syncthreads();
  bf16_t* out = static_cast<bf16_t*>(which == 0 ? a.Q_out : a.pages);
  // thread: one chunk of every kStep-th row; four rows' LDS reads in flight together
  constexpr int kStep = kRingThreads / (16 * kHeads);
  const int c = tid % (16 * kHeads), t0 = tid / (16 * kHeads);
  const int64_t* dst_of = sm_dst + (c >> 4) * kTok;
#pragma unroll 4
  for (int k = 0; k < kTok / kStep; ++k) {
    const int t = t0 + kStep * k;
    const uint4 piece = *reinterpret_cast<const uint4*>(sO + t * (128 * kHeads) + ((c ^ (t & 15)) * 8));
    const int64_t dst = dst_of[t];
    if (dst >= 0) *reinterpret_cast<uint4*>(out + dst + (c & 15) * 8) = piece;
  }
}

// generic path: thread = (compacted row, which of Q/K/V, head, rotary pair i)
template <typename T>
__global__ __launch_bounds__(256) void qkv_generic_kernel(QkvArgs a, RopeTableD rt) {
  const int r = blockIdx.x;
  const int total = a.off[a.B];
  if (r == 0 && blockIdx.y == 0) set_lengths(a, threadIdx.x, blockDim.x);
  if (r >= total) return;
  const int half = a.Dh / 2, H = a.H, Dh = a.Dh;
  const int e = blockIdx.y * blockDim.x + threadIdx.x;  // pair index over 3 * H * half
  if (e >= 3 * H * half) return;
  const int which = e / (H * half), head = (e / half) % H, i = e % half;
  const T* x = static_cast<const T*>(a.x) + static_cast<int64_t>(r) * a.ldx;
  const T* w0 = static_cast<const T*>(a.W[which]) + (static_cast<int64_t>(head) * Dh + i) * a.d;
  const T* w1 = w0 + static_cast<int64_t>(half) * a.d;
  float s0 = 0.f, s1 = 0.f;
  for (int64_t c = 0; c < a.d; ++c) {
    const float xv = Elem<T>::load(x + c);
    s0 = fmaf(xv, Elem<T>::load(w0 + c), s0);
    s1 = fmaf(xv, Elem<T>::load(w1 + c), s1);
  }
  if (which < 2 && a.pos) {
    const double ang = static_cast<double>(a.pos[r]) * rt.f[i];
    const float cs = static_cast<float>(cos(ang)), sn = static_cast<float>(sin(ang));
    const float y0 = s0 * cs - s1 * sn, y1 = s1 * cs + s0 * sn;
    s0 = y0;
    s1 = y1;
  }
  T* out;
  if (which == 0) {
    out = static_cast<T*>(a.Q_out) + (static_cast<int64_t>(r) * H + head) * Dh;
  } else {
    const int b = seq_of_row(a.off, a.B, r);
    int64_t dst = page_slot(a, b, r - a.off[b], head);
    if (dst < 0) return;
    if (which == 2) dst += static_cast<int64_t>(H) * kPage * Dh;
    out = static_cast<T*>(a.pages) + dst;
  }
  Elem<T>::store(out + i, s0);
  Elem<T>::store(out + i + half, s1);
}

template <typename T>
int launch_generic(const QkvArgs& a, int64_t rows, double base, hipStream_t st) {
  RopeTableD rt{};
  for (int i = 0; i < a.Dh / 2; ++i) rt.f[i] = base > 0 ? pow(base, -2.0 * i / a.Dh) : 0.0;
  const int pairs = 3 * a.H * (a.Dh / 2);
  dim3 grid(static_cast<unsigned>(rows), static_cast<unsigned>(ceil_div(pairs, 256)));
  hipLaunchKernelGGL(qkv_generic_kernel<T>, grid, dim3(256), 0, st, a, rt);
  DLLAVA_CHECK_LAUNCH("qkv_generic_kernel");
  return DLLAVA_OK;
}

// returns 1 if the shape is not handled by the matrix-core kernel
int launch_mfma(const QkvArgs& a, int64_t rows, double base, hipStream_t st) {
  if (a.Dh != 128 || a.d % 64 != 0 || a.ldx % 8 != 0) return 1;
  RopeTable rt{};
  const double two_pi = 6.283185307179586476925287;
  for (int i = 0; i < 64; ++i) {
    const double rev = base > 0 ? pow(base, -2.0 * i / 128.0) / two_pi : 0.0;
    rt.hi[i] = static_cast<float>(rev);
    rt.lo[i] = static_cast<float>(rev - static_cast<double>(rt.hi[i]));
  }
  // The tile that takes least: few rows want the tiles of one head, which leave less of the chip idle (32 heads, d = 4096,
  // this pick / the best tile of two heads: 107 rows 22 / 46 us, 214 rows 31 / 47, 350 rows 41 / 48, 1000 rows the latter,
  // 83 us).  Lane offsets into the whole of a matrix and of x are 32-bit in the tiles of two heads.
  const int forced = launch_override(DLLAVA_LAUNCH_QKV_TILE);
  auto heads_tiles = [&](const RingTile& c) -> int64_t { return 3 * ceil_div(a.H, c.fi / 4); };
  const RingTile* t = ring_pick(a.d, forced == 1 ? 3 : forced, [&](const RingTile& c) -> int64_t {
    if (c.per_cu > 1 || c.fi < 4) return 0;
    const bool fits = static_cast<int64_t>(a.H) * 128 * a.d * 2 < (int64_t{1} << 32) && rows * a.ldx * 2 < (int64_t{1} << 32);
    const int64_t n = ceil_div(rows, 32 * c.jt) * heads_tiles(c);
    return (c.fi == 8 && !fits) || n > 0x7fffffffLL - 8 ? 0 : n;
  });
  if (!t) return 1;
  const int n_ft = static_cast<int>(heads_tiles(*t));
  const int64_t per_xcd = ceil_div(n_ft * ceil_div(rows, 32 * t->jt), kRingXcds);
  const dim3 grid(static_cast<unsigned>(per_xcd * kRingXcds)), block(kRingThreads);
  switch (t->id) {
    case 10: hipLaunchKernelGGL((qkv_ring_kernel<4, 2>), grid, block, 0, st, a, rt, n_ft); break;
    case 3: hipLaunchKernelGGL((qkv_ring_kernel<4, 4>), grid, block, 0, st, a, rt, n_ft); break;
    case 9: hipLaunchKernelGGL((qkv_ring_kernel<4, 6>), grid, block, 0, st, a, rt, n_ft); break;
    case 4: hipLaunchKernelGGL((qkv_ring_kernel<8, 4>), grid, block, 0, st, a, rt, n_ft); break;
    case 5: hipLaunchKernelGGL((qkv_ring_kernel<8, 5>), grid, block, 0, st, a, rt, n_ft); break;
    case 6: hipLaunchKernelGGL((qkv_ring_kernel<8, 6>), grid, block, 0, st, a, rt, n_ft); break;
    case 7: hipLaunchKernelGGL((qkv_ring_kernel<8, 7>), grid, block, 0, st, a, rt, n_ft); break;
    default: hipLaunchKernelGGL((qkv_ring_kernel<8, 8>), grid, block, 0, st, a, rt, n_ft); break;
  }
  DLLAVA_CHECK_LAUNCH("qkv_ring_kernel");
  return DLLAVA_OK;
}

}  // namespace

}  // namespace dllava

using namespace dllava;

extern "C" int dllava_qkv_project(const void* x, int64_t ldx, int64_t rows, int64_t d,
                                  int32_t B, const int32_t* off, const int32_t* pos,
                                  const void* Wq, const void* Wk, const void* Wv, float rope_base,
                                  void* Q_out, const dllava_kv_cache* cache, int32_t* err_flag,
                                  int dtype, void* stream) {
  DLLAVA_REQUIRE(B >= 0 && rows >= 0, DLLAVA_EINVAL, "qkv_project: B = %d, rows = %lld", B, (long long)rows);
  DLLAVA_REQUIRE(rows <= 0x7fffffffLL, DLLAVA_ESHAPE, "qkv_project: rows must fit in int32");
  DLLAVA_REQUIRE(dtype == DLLAVA_F32 || dtype == DLLAVA_BF16, DLLAVA_EDTYPE, "qkv_project: unknown dtype %d", dtype);
  if (int rc = check_cache(cache, "qkv_project")) return rc;
  DLLAVA_REQUIRE(cache->dtype == dtype, DLLAVA_EDTYPE, "qkv_project: cache dtype differs from the call's");
  DLLAVA_REQUIRE(d > 0 && ldx >= d, DLLAVA_EINVAL, "qkv_project: d = %lld, ldx = %lld", (long long)d, (long long)ldx);
  const int64_t esz = dtype == DLLAVA_BF16 ? 2 : 4;
  DLLAVA_REQUIRE((d * esz) % 16 == 0 && (ldx * esz) % 16 == 0, DLLAVA_ESHAPE,
                 "qkv_project: rows of x and of the weights must be multiples of 16 bytes");
  DLLAVA_REQUIRE(rope_base == rope_base && rope_base < INFINITY, DLLAVA_EINVAL, "qkv_project: bad rope_base");
  if (B == 0 || rows == 0) return DLLAVA_OK;
  DLLAVA_REQUIRE(x && off && Wq && Wk && Wv && Q_out, DLLAVA_ENULL, "qkv_project: x, off, Wq, Wk, Wv and Q_out are required");
  DLLAVA_REQUIRE(rope_base <= 0.f || pos, DLLAVA_ENULL, "qkv_project: pos is required when rope_base > 0");
  DLLAVA_REQUIRE(aligned(x, 16) && aligned(Wq, 16) && aligned(Wk, 16) && aligned(Wv, 16) && aligned(Q_out, 16),
                 DLLAVA_EINVAL, "qkv_project: x, Wq, Wk, Wv, Q_out must be 16-byte aligned");

  QkvArgs a{};
  a.x = x; a.ldx = ldx; a.d = d; a.B = B; a.off = off; a.pos = rope_base > 0.f ? pos : nullptr;
  a.W[0] = Wq; a.W[1] = Wk; a.W[2] = Wv;
  a.H = cache->H; a.Dh = cache->Dh; a.Q_out = Q_out;
  a.pages = cache->pages; a.block_table = cache->block_table; a.cache_len = cache->cache_len;
  a.max_pages = cache->max_pages_per_seq; a.err_flag = err_flag;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == DLLAVA_BF16) {
    const int rc = launch_mfma(a, rows, rope_base, st);
    if (rc <= 0) return rc;
    return launch_generic<bf16_t>(a, rows, rope_base, st);
  }
  return launch_generic<float>(a, rows, rope_base, st);
}
