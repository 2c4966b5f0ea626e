// Matrix-core predictor scoring for bfloat16 inputs (Eq. 5 line 1 / Eq. 11 line 1 of the paper):
//   D = GELU(x W1^T + b1) W2^T + b2,   x [M,d], W1 [dh,d], W2 [2,dh].
//
// Both kernels compute the TRANSPOSED product  A^T = W1 . x^T  (hidden units down the rows, tokens
// across the columns).  x and W1 are both contiguous along d, so either operand fragment is one 16-byte
// load per lane, and in the MFMA result layout a lane then holds many hidden units of ONE token: bias,
// GELU and the 2-way logit contraction over hidden units happen in registers, the pre-activations never
// leave the chip, and only one cross-lane step (lanes l and l+32, or l+16/l+32/l+48) is left.
//
//  * score_ring_kernel   (M > 64, prefill): tiles of 128 or 256 units x 64 .. 256 tokens on the products of gemm_ring.h.
//    Each block leaves a partial logit pair per token; the last block of a token tile (device-scope counter) adds the
//    partials in tile order and the bias.
//  * score_splitk_kernel (M <= 64, decode: one row per sequence): W1 read once, cut over units and d; see
//    score_splitk.h.
// All reductions run in a fixed order: results are bit-reproducible.  The counters of the two forms live in
// disjoint regions at the start of the workspace (layout in score_splitk.h), start at zero and are returned to
// zero by the block that consumes them, so one workspace serves calls of either form in any order.
#include "gemm_ring.h"
#include "score_splitk.h"

namespace dllava {

namespace {

constexpr int kMaxCounters = static_cast<int>(kGemmCntBytes / sizeof(int32_t));  // one per token tile

// ------------------------------------------------------------------------------------------------
// GEMM for many rows: 32*FI units x 32*JB tokens per block, one block per compute unit (gemm_ring.h)
// ------------------------------------------------------------------------------------------------
// Each block leaves a partial logit pair per token; the last block of a token tile (device-scope counter) adds the partials
// of the unit tiles in tile order and the bias.  Wave w holds units 16*FI*(w/2) + [0, 16*FI) of the unit tile for half of
// the 32*JB tokens of the token tile.  The tile is chosen on the host (ring_pick).
template <int FI, int JB>
__global__ __launch_bounds__(kRingThreads, 1) void score_ring_kernel(ScoreArgs a, int32_t* counters, float* partial,
                                                                     int n_ut, int n_mt, int per_xcd) {
  constexpr int kTok = 32 * JB, kUnits = 32 * FI;
  constexpr int kDepth = kRingLdsBytes / ((FI + JB) * 32 * kRingRowBytes);  // FI < 8: stages that LDS holds
  __shared__ __align__(1024) char smem_raw[kRingLdsBytes];
  DLLAVA_LDS char* smem = (DLLAVA_LDS char*)smem_raw;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  int ut, mt;
  if (!ring_tile(n_ut, n_mt, per_xcd, ut, mt)) return;
  const int64_t M = a.M, d = a.d, dh = a.dh;

  // this lane's tile loads: byte offsets from W1 / x (rows past the end repeat the last row: their units count as
  // zero, their tokens are not written)
  std::conditional_t<FI == 8, uint32_t, int64_t> ga[FI];
  int64_t gb[JB];  // gathered rows of x may lie far apart
#pragma unroll
  for (int j = 0; j < FI; ++j) {
    const int row = ring_load_row(w, j, lane);
    int64_t u = static_cast<int64_t>(ut) * kUnits + row;
    if (u >= dh) u = dh - 1;
    ga[j] = static_cast<decltype(+ga[0])>(u * d * 2) + ring_load_chunk_bytes(row, lane);
  }
  // gathered spans: the row mapping from a table in the (not yet used) ring memory
  SpanTable* spans = reinterpret_cast<SpanTable*>(smem_raw);
  const bool use_table = a.seq_off != nullptr && a.B > 0 && a.B <= kSpanLdsMax;
  if (use_table) span_table_build<kRingThreads>(spans, a.seq_off, a.vis_start, a.vis_len, a.B);
  const int64_t m_first = static_cast<int64_t>(mt) * kTok, m_last = m_first + kTok <= M ? m_first + kTok - 1 : M - 1;
  int64_t m_of[JB], src[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    m_of[j] = m_first + ring_load_row(w, j, lane);
    if (m_of[j] >= M) m_of[j] = M - 1;
  }
  int64_t rows_in_spans;
  if (use_table) {
    rows_in_spans = spans->prefix[a.B];
#pragma unroll
    for (int j = 0; j < JB; ++j) src[j] = span_table_row(spans, a.B, m_of[j]);
  } else {
    rows_in_spans = score_src_rows<JB>(a.seq_off, a.vis_start, a.vis_len, a.B, m_first, m_last, m_of, src);
  }
#pragma unroll
  for (int j = 0; j < JB; ++j)
    gb[j] = (src[j] < 0 ? 0 : src[j]) * a.ldx * 2 + ring_load_chunk_bytes(ring_load_row(w, j, lane), lane);
  if (use_table) __syncthreads();  // the tile loads overwrite the table
  ring_f32x4 acc[FI][JB];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) acc[i][j] = ring_f32x4{0.f, 0.f, 0.f, 0.f};
  const char *Ab = static_cast<const char*>(a.W1), *Bb = static_cast<const char*>(a.x);
  if constexpr (FI == 8)
    gemm_ring_halves<FI, JB>(Ab, ga, Bb, gb, static_cast<int>(d / kRingBK), smem, w, acc);
  else
    gemm_ring_small<FI, JB, kDepth>(Ab, ga, Bb, gb, static_cast<int>(d / kRingBK), smem, w, acc);

  // epilogue: lane holds, for token 16*JB*(w%2) + 16*j + lane%16, units 16*FI*(w/2) + 16*i + 4*(lane/16) + 0..3
  const bf16_t* W2 = static_cast<const bf16_t*>(a.W2);
  const bool has_b1 = a.b1 != nullptr;
  const bf16_t* zero16 = reinterpret_cast<const bf16_t*>(kZeroWords);
  float p[JB][2];
#pragma unroll
  for (int j = 0; j < JB; ++j) p[j][0] = p[j][1] = 0.f;
  // bias and the two weights of the lane's units, all requested at once; with dh a multiple of 4 (and aligned vectors)
  // whole quadruples of units exist or do not, one load each
  const bool quads = dh % 4 == 0 && (reinterpret_cast<uintptr_t>(W2) % 8 == 0) && (reinterpret_cast<uintptr_t>(a.b1) % 16 == 0);
  float4 bq[FI];
  uint2 q0[FI], q1[FI];
  const int units = static_cast<int>(dh), u_lane = ut * kUnits + 16 * FI * (w >> 1) + 4 * (lane >> 4);  // dh <= 2^20
  if (quads) {
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const int u0 = u_lane + 16 * i;
      const bool ok = u0 < units;  // operands that must be zero come from kZeroWords: no load under a condition
      bq[i] = *reinterpret_cast<const float4*>((ok & has_b1) ? a.b1 + u0 : kZeroWords);
      q0[i] = *reinterpret_cast<const uint2*>(ok ? W2 + u0 : zero16);
      q1[i] = *reinterpret_cast<const uint2*>(ok ? W2 + dh + u0 : zero16);
    }
  } else {  // through the ring memory, one thread per unit
    __syncthreads();
    float* sb = reinterpret_cast<float*>(smem_raw);
    bf16_t* s0 = reinterpret_cast<bf16_t*>(sb + kUnits);
    bf16_t* s1 = s0 + kUnits;
    if (tid < kUnits) {
      const int u = ut * kUnits + tid;
      const bool ok = u < units;
      sb[tid] = ok && has_b1 ? a.b1[u] : 0.f;
      s0[tid] = ok ? W2[u] : bf16_t{0};
      s1[tid] = ok ? W2[dh + u] : bf16_t{0};
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const int at = u_lane - ut * kUnits + 16 * i;
      bq[i] = *reinterpret_cast<const float4*>(sb + at);
      q0[i] = *reinterpret_cast<const uint2*>(s0 + at);
      q1[i] = *reinterpret_cast<const uint2*>(s1 + at);
    }
  }
#pragma unroll
  for (int i = 0; i < FI; ++i) {
#pragma unroll
    for (int j = 0; j < JB; ++j) ring_tie_acc(acc[i][j]);  // in accumulation registers until here: the others do not hold them all
    const float bias[4] = {bq[i].x, bq[i].y, bq[i].z, bq[i].w};
    const float w20[4] = {bf16lo_to_f32(q0[i].x), bf16hi_to_f32(q0[i].x), bf16lo_to_f32(q0[i].y), bf16hi_to_f32(q0[i].y)};
    const float w21[4] = {bf16lo_to_f32(q1[i].x), bf16hi_to_f32(q1[i].x), bf16lo_to_f32(q1[i].y), bf16hi_to_f32(q1[i].y)};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // past dh the last unit repeats: its weight of zero alone would make NaN of an infinite value
      uint32_t real = u_lane + 16 * i + r < units ? ~0u : 0u;
      asm("" : "+v"(real));  // of a choice it knows the compiler makes a branch around every GELU
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const float g = __uint_as_float(__float_as_uint(gelu_erf_fast(acc[i][j][r] + bias[r])) & real);
        p[j][0] = fmaf(g, w20[r], p[j][0]);
        p[j][1] = fmaf(g, w21[r], p[j][1]);
      }
#pragma unroll
      for (int j = 0; j < JB; ++j) asm volatile("" : "+v"(p[j][0]), "+v"(p[j][1]));  // summed here: the compiler kept all values to sum them at the end
      __builtin_amdgcn_sched_barrier(0);  // JB values at a time: the accumulators leave no registers for more
    }
  }
  // the ring memory becomes the waves' partial sums: every wave has drained its own tile loads, the barrier covers
  // the others'
  __syncthreads();
  float* sm_p = reinterpret_cast<float*>(smem_raw);  // [2 halves of the units][kTok][2]
  int* sm_last = reinterpret_cast<int*>(smem_raw + 2 * kTok * 2 * sizeof(float));
#pragma unroll
  for (int j = 0; j < JB; ++j) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      p[j][c] += __shfl_xor(p[j][c], 16, kWave);
      p[j][c] += __shfl_xor(p[j][c], 32, kWave);
    }
    if (lane < 16) {
      const int t = 16 * JB * (w & 1) + 16 * j + lane;
      sm_p[((w >> 1) * kTok + t) * 2 + 0] = p[j][0];
      sm_p[((w >> 1) * kTok + t) * 2 + 1] = p[j][1];
    }
  }
  __syncthreads();
  for (int t = tid; t < 2 * kTok; t += kRingThreads) {
    const int tok = t >> 1, c = t & 1;
    const int64_t m = static_cast<int64_t>(mt) * kTok + tok;
    const float v = sm_p[tok * 2 + c] + sm_p[(kTok + tok) * 2 + c];
    if (m < M) st_agent(partial + (static_cast<size_t>(ut) * M + m) * 2 + c, v);
  }
  block_publish();
  if (tid == 0) *sm_last = (add_agent(&counters[mt % kMaxCounters], 1) == n_ut - 1);
  __syncthreads();
  if (!*sm_last) return;
  for (int t = tid; t < 2 * kTok; t += kRingThreads) {
    const int tok = t >> 1, c = t & 1;
    const int64_t m = static_cast<int64_t>(mt) * kTok + tok;
    if (m < M && m < rows_in_spans) {
      float s = a.b2 ? a.b2[c] : 0.f;
      for (int t0 = 0; t0 < n_ut; t0 += 8) {  // independent loads in flight, then a fixed-order sum
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          v[u] = (t0 + u < n_ut) ? ld_agent(partial + (static_cast<size_t>(t0 + u) * M + m) * 2 + c) : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
      }
      a.logits[2 * m + c] = s;
    }
  }
  if (tid == 0) zero_agent(&counters[mt % kMaxCounters]);
}

template <int FI, int JB>
int score_ring_launch(const ScoreArgs& a, int32_t* counters, float* partial, hipStream_t st) {
  const int64_t n_mt = ceil_div(a.M, 32 * JB), n_ut = ceil_div(a.dh, 32 * FI);
  const int64_t per_xcd = ceil_div(n_mt * n_ut, kRingXcds);
  hipLaunchKernelGGL((score_ring_kernel<FI, JB>), dim3(static_cast<unsigned>(per_xcd * kRingXcds)), dim3(kRingThreads), 0, st, a, counters,
                     partial, static_cast<int>(n_ut), static_cast<int>(n_mt), static_cast<int>(per_xcd));
  DLLAVA_CHECK_LAUNCH("score_ring_kernel");
  return DLLAVA_OK;
}

}  // namespace

size_t score_mfma_workspace(int64_t M, int64_t d, int64_t dh) {
  // Non-decreasing in M, so a workspace sized for the largest row count serves every smaller one: the split-K form
  // of at most 64 rows needs more than the GEMM form of a few hundred.
  const size_t small = round_up(split_workspace(M < 64 ? M : 64, d, dh), 256);
  if (M <= 64) return small;
  const size_t part = static_cast<size_t>(ceil_div(dh, 128)) * M * 2 * sizeof(float);
  const size_t gemm = kScoreScratchOffset + round_up(part, 256);
  return gemm > small ? gemm : small;
}

// returns 1 if the shape is not handled here
int score_mfma_launch(const ScoreArgs& a, hipStream_t st) {
  if (a.d % 64 != 0 || a.ldx % 8 != 0) return 1;
  int32_t* counters = reinterpret_cast<int32_t*>(static_cast<char*>(a.workspace) + kSpAccBytes + kSpCntBytes);
  float* partial = reinterpret_cast<float*>(static_cast<char*>(a.workspace) + kScoreScratchOffset);
  if (a.M <= 64) {
    if (a.seq_off) return 1;  // span gathering is only wired into the GEMM path
    const SplitPlan p = split_plan(a.d, a.dh);
    if (p.G > kSpMaxGroups) return 1;
    const dim3 grid(static_cast<unsigned>(p.G * p.KS)), block(kSpThreads);
    if (a.M <= 16)
      hipLaunchKernelGGL(score_splitk_kernel<1>, grid, block, 0, st, a, p.G, p.KS, p.ppb);
    else if (a.M <= 32)
      hipLaunchKernelGGL(score_splitk_kernel<2>, grid, block, 0, st, a, p.G, p.KS, p.ppb);
    else
      hipLaunchKernelGGL(score_splitk_kernel<4>, grid, block, 0, st, a, p.G, p.KS, p.ppb);
    DLLAVA_CHECK_LAUNCH("score_splitk_kernel");
    return DLLAVA_OK;
  }
  // Many rows.  The tile that takes least: few rows want the tiles of 128 units, which leave less of the chip idle (d = 4096,
  // dh = 1024, this pick / the best tile of 256 units: 576 rows 22 / 48 us, 2880 rows 34 / 50, 5760 rows 48 / 52, 11520 rows
  // the latter, 77 us).  Every token tile needs its own counter, the workspace holds partials of unit tiles of 128 or more,
  // and lane offsets into the 256 rows of a large W1 tile are 32-bit.
  const int forced = launch_override(DLLAVA_LAUNCH_SCORE_TILE);
  const RingTile* t = ring_pick(a.d, forced == 1 ? 3 : forced, [&](const RingTile& c) -> int64_t {
    const int64_t n_mt = ceil_div(a.M, 32 * c.jt), n = n_mt * ceil_div(a.dh, 32 * c.fi);
    if (c.per_cu > 1 || c.fi < 4 || n_mt > kMaxCounters || n > 0x7fffffffLL - 8) return 0;
    return c.fi == 8 && a.dh * a.d * 2 >= (int64_t{1} << 32) ? 0 : n;
  });
  if (!t) return 1;
  switch (t->id) {
    case 10: return score_ring_launch<4, 2>(a, counters, partial, st);
    case 3: return score_ring_launch<4, 4>(a, counters, partial, st);
    case 9: return score_ring_launch<4, 6>(a, counters, partial, st);
    case 4: return score_ring_launch<8, 4>(a, counters, partial, st);
    case 5: return score_ring_launch<8, 5>(a, counters, partial, st);
    case 6: return score_ring_launch<8, 6>(a, counters, partial, st);
    case 7: return score_ring_launch<8, 7>(a, counters, partial, st);
    default: return score_ring_launch<8, 8>(a, counters, partial, st);
  }
}

}  // namespace dllava
