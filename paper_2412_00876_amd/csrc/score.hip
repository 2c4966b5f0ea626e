// dllava_score: predictor logits D = GELU(x W1^T + b1) W2^T + b2 (Eq. 5 line 1 / Eq. 11 line 1 of the
// paper, with the two-layer predictor d -> dh -> 2).
//
// Precision-generic path, for float32 inputs and shapes the matrix-core kernels do not cover.  A block takes R scored
// rows (1 or 4: W1 is read once per block), staged in LDS as float32.  Each of its waves takes 1 to 8 hidden units at a
// time, its lanes strided over d with 16-byte loads of those W1 rows, the next loads in flight while the last are
// multiplied -- the first ones before the rows are staged, which they do not depend on.
// The sums of a wave's units are reduced together: at each exchange a lane hands over half of its sums and keeps the
// other half, so eight units cost ten lane exchanges instead of 48, and bias and GELU are applied to all of them at once.
// All sums run in a fixed order: bit-reproducible.
// What bounds it is the chain of these steps for few rows, the LDS and L1 reads of the multiply for many.  float32,
// d = 512, dh = 128, with four waves and one unit per wave at a time / now: one row 19.8 / 4.7 us, 200 rows 20.9 / 5.4 us,
// 4608 rows 104 / 32 us; d = 4096, dh = 512: one row 591 / 77 us, 4608 rows 2195 / 581 us.  The form follows dh and M, see
// launch_generic.
#include "score_args.h"

namespace dllava {

namespace {

// kUnits: hidden units a wave takes at a time; kWaves: waves of a block
template <typename T, int R, int kUnits, int kWaves>
__global__ __launch_bounds__(kWaves* kWave) void score_generic_kernel(ScoreArgs a) {
  constexpr int kThreads = kWaves * kWave;
  extern __shared__ float xs[];  // [R][d]
  __shared__ float sm_l[kWaves][R][2];
  constexpr int E = Elem<T>::kPer16B;
  constexpr int kPerUnit = kWave / kUnits;
  const int64_t m0 = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * R;
  if (m0 >= a.M) return;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int d = static_cast<int>(a.d), chunks = d / E, dh = static_cast<int>(a.dh);
  const T* W1 = static_cast<const T*>(a.W1);
  const T* W2 = static_cast<const T*>(a.W2);
  // piece (j0, c): chunk c of units j0 .. j0+7 (units past dh repeat the last one and count as zero; chunks past the row
  // repeat the last one and are not used)
  uint4 wv[kUnits];
  auto load = [&](int j0, int c) __attribute__((always_inline)) {
    const int cc = c < chunks ? c : chunks - 1;
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const int j = j0 + u < dh ? j0 + u : dh - 1;
      wv[u] = *reinterpret_cast<const uint4*>(W1 + static_cast<int64_t>(j) * d + static_cast<int64_t>(cc) * E);
    }
  };
  constexpr bool kAhead = kUnits > 2;  // with one or two units the loop is left to the compiler, which has several pieces in flight
  if constexpr (kAhead) load(w * kUnits, lane);
  int64_t src[R], m_of[R];
#pragma unroll
  for (int r = 0; r < R; ++r) m_of[r] = m0 + r < a.M ? m0 + r : a.M - 1;
  score_src_rows<R>(a.seq_off, a.vis_start, a.vis_len, a.B, m0, m_of[R - 1], m_of, src);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (m0 + r >= a.M) src[r] = -1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (src[r] < 0) continue;  // beyond the spans: not read, not written
    const T* xrow = static_cast<const T*>(a.x) + src[r] * a.ldx;
    for (int c = tid; c < chunks; c += kThreads) {
      float f[E];
      Elem<T>::unpack(*reinterpret_cast<const uint4*>(xrow + static_cast<int64_t>(c) * E), f);
#pragma unroll
      for (int e = 0; e < E; ++e) xs[r * d + c * E + e] = f[e];
    }
  }
  __syncthreads();
  float l0[R], l1[R];
#pragma unroll
  for (int r = 0; r < R; ++r) l0[r] = l1[r] = 0.f;
  for (int j0 = w * kUnits; j0 < dh; j0 += kWaves * kUnits) {
    const int j = j0 + lane / kPerUnit;  // the unit whose whole sum this lane ends with
    const bool ok = j < dh;
    const float bias = ok && a.b1 ? a.b1[j] : 0.f;
    const float w20 = ok ? Elem<T>::load(W2 + j) : 0.f, w21 = ok ? Elem<T>::load(W2 + a.dh + j) : 0.f;
    float acc[R][kUnits];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int u = 0; u < kUnits; ++u) acc[r][u] = 0.f;
    auto multiply = [&](const uint4 (&piece)[kUnits], int c) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kUnits; ++u) {
        float f[E];
        Elem<T>::unpack(piece[u], f);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < E; ++e) acc[r][u] = fmaf(xs[r * d + c * E + e], f[e], acc[r][u]);
      }
    };
    if constexpr (!kAhead) {
      for (int c = lane; c < chunks; c += kWave) {
        load(j0, c);
        multiply(wv, c);
      }
    } else {
      for (int c0 = 0; c0 < chunks; c0 += kWave) {  // wave-uniform
        const int c = c0 + lane;
        uint4 cur[kUnits];
#pragma unroll
        for (int u = 0; u < kUnits; ++u) cur[u] = wv[u];
        if (c0 + kWave < chunks)
          load(j0, c + kWave);
        else if (j0 + kWaves * kUnits < dh)
          load(j0 + kWaves * kUnits, lane);
        if (c < chunks) multiply(cur, c);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float* v = acc[r];
#pragma unroll
      for (int half = kUnits / 2, o = 32; half >= 1; half >>= 1, o >>= 1) {
        const bool up = (lane & o) != 0;
#pragma unroll
        for (int u = 0; u < half; ++u) {
          const float give = up ? v[u] : v[u + half], keep = up ? v[u + half] : v[u];
          v[u] = keep + __shfl_xor(give, o, kWave);
        }
      }
      float sum = v[0];
#pragma unroll
      for (int o = kPerUnit / 2; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, kWave);
      const float g = ok ? gelu_erf(sum + bias) : 0.f;  // a weight of zero alone would make NaN of an infinite repeat
      l0[r] = fmaf(g, w20, l0[r]);
      l1[r] = fmaf(g, w21, l1[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int o = kPerUnit; o < kWave; o <<= 1) {  // over the wave's units (the lanes of a unit hold the same)
      l0[r] += __shfl_xor(l0[r], o, kWave);
      l1[r] += __shfl_xor(l1[r], o, kWave);
    }
    if (lane == 0) {
      sm_l[w][r][0] = l0[r];
      sm_l[w][r][1] = l1[r];
    }
  }
  __syncthreads();
  if (tid < 2 * R) {
    const int r = tid >> 1, c = tid & 1;
    float s = a.b2 ? a.b2[c] : 0.f;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) s += sm_l[i][r][c];
    int64_t mine = -1;
#pragma unroll
    for (int q = 0; q < R; ++q) mine = q == r ? src[q] : mine;
    if (mine >= 0) a.logits[2 * (m0 + r) + c] = s;
  }
}

template <typename T, int R, int kUnits, int kWaves>
void launch_form(const ScoreArgs& a, hipStream_t st) {
  const int64_t n = ceil_div(a.M, R);
  const int64_t gx = n < (1 << 20) ? n : (1 << 20);  // a grid dimension holds fewer than 2^32 threads
  const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(ceil_div(n, gx)));
  hipLaunchKernelGGL((score_generic_kernel<T, R, kUnits, kWaves>), grid, dim3(kWaves * kWave), R * static_cast<size_t>(a.d) * sizeof(float), st, a);
}

// Which form.  As many waves and units per wave as there are units for, up to 16 and 8; a row whose units are few is cheap
// and wants many small blocks in flight instead (one row, float32, d = 512, waves x units: dh = 4 2.5 us at 4x1 against 4.3
// at 16x8, dh = 16 3.0 at 4x4 against 4.5, dh = 32 3.1 at 8x4 against 4.6, dh = 48 4.0 at 8x4 against 4.6; 20000 rows,
// dh = 2: 19 us at 4x1, 92 at 16x4).  A compute unit holds one block of 16 waves at a time, so more than 256 rows singly go
// two to a compute unit with 8 waves (float32 / bfloat16, dh = 128, 500 rows: 9.1 / 11.1 us against 11.6 / 12.9), and above
// 512 rows, a third round, a block takes four of them (500 rows that way: 10.8 / 16.1; 600 rows 11.0 / 16.4 against 11.2 /
// 16.8 with 8 waves), with four waves of eight units from the second round of those blocks on (1000 rows 14.7 us against
// 11.0 with 16 waves, 2000 rows 16.2 against 20.9).  Four float32 rows have to fit 64 KiB of LDS.
template <typename T>
int launch_generic(const ScoreArgs& a, hipStream_t st) {
  const bool four = a.M > 512 && 4 * a.d * static_cast<int64_t>(sizeof(float)) <= 64 * 1024;
  if (a.dh <= 4)
    launch_form<T, 1, 1, 4>(a, st);
  else if (a.dh <= 8)
    launch_form<T, 1, 2, 4>(a, st);
  else if (a.dh <= 16)
    launch_form<T, 1, 4, 4>(a, st);
  else if (four && a.M > 1024)
    launch_form<T, 4, 8, 4>(a, st);
  else if (four)
    launch_form<T, 4, 4, 16>(a, st);
  else if (a.M > 256 || a.dh <= 32)
    launch_form<T, 1, 4, 8>(a, st);
  else
    launch_form<T, 1, sizeof(T) == 4 ? 8 : 4, 16>(a, st);  // the units that the registers of 16 waves hold
  DLLAVA_CHECK_LAUNCH("score_generic_kernel");
  return DLLAVA_OK;
}

}  // namespace

}  // namespace dllava

using namespace dllava;

extern "C" size_t dllava_score_workspace(int64_t M, int64_t d, int64_t dh, int dtype) {
  if (dtype != DLLAVA_BF16 || M <= 0) return 256;
  return score_mfma_workspace(M, d, dh) + 256;
}

extern "C" int dllava_score(const void* x, int64_t ldx, int64_t M, int32_t B, const int32_t* seq_off,
                            const int32_t* vis_start, const int32_t* vis_len, int64_t d, int64_t dh,
                            const void* W1, const float* b1, const void* W2, const float* b2, int dtype,
                            float* logits, void* workspace, size_t workspace_bytes, void* stream) {
  DLLAVA_REQUIRE(dtype == DLLAVA_F32 || dtype == DLLAVA_BF16, DLLAVA_EDTYPE, "score: unknown dtype %d", dtype);
  DLLAVA_REQUIRE(M >= 0 && M <= 0x7fffffffLL, DLLAVA_ESHAPE, "score: bad M = %lld", (long long)M);
  DLLAVA_REQUIRE(d > 0 && d % 8 == 0 && d <= 16384, DLLAVA_ESHAPE, "score: d must be a multiple of 8, at most 16384 (got %lld)",
                 (long long)d);
  DLLAVA_REQUIRE(dh >= 1 && dh <= (1 << 20), DLLAVA_ESHAPE, "score: bad dh = %lld", (long long)dh);
  DLLAVA_REQUIRE(ldx >= d && (ldx * dtype_size(dtype)) % 16 == 0, DLLAVA_ESHAPE,
                 "score: ldx must be >= d and keep rows 16-byte aligned (got %lld)", (long long)ldx);
  if (M == 0) return DLLAVA_OK;
  DLLAVA_REQUIRE(x && W1 && W2 && logits, DLLAVA_ENULL, "score: x, W1, W2, logits are required");
  DLLAVA_REQUIRE(aligned(x, 16) && aligned(W1, 16), DLLAVA_EINVAL, "score: x and W1 must be 16-byte aligned");
  if (seq_off) {
    DLLAVA_REQUIRE(vis_start && vis_len, DLLAVA_ENULL, "score: vis_start and vis_len go with seq_off");
    DLLAVA_REQUIRE(B > 0, DLLAVA_EINVAL, "score: B must be positive when seq_off is given");
  }
  const size_t need = dllava_score_workspace(M, d, dh, dtype);
  DLLAVA_REQUIRE(workspace && aligned(workspace, 256) && workspace_bytes >= need, DLLAVA_EWORKSPACE,
                 "score: workspace needs %zu bytes, 256-byte aligned (got %zu)", need, workspace_bytes);

  ScoreArgs a{x, ldx, M, d, dh, B, seq_off, vis_start, vis_len, W1, b1, W2, b2, logits, workspace};
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == DLLAVA_BF16) {
    const int rc = score_mfma_launch(a, st);
    if (rc <= 0) return rc;
    return launch_generic<bf16_t>(a, st);
  }
  return launch_generic<float>(a, st);
}
