// Matrix-core attention of long sequences, bfloat16: causal over the reduced prefill set (Eq. 1 of the paper applied to
// S^{P*}), keys and values in pages or in rows, and unmasked within spans (the image predictor's blocks).  The kernel's body
// and what bounds it: attn_tiles.h.
#include "attn_tiles.h"

namespace dllava {

namespace {

template <int DH, int NWQ, Mode MODE>
__global__ __launch_bounds__(NWQ * kWave, NWQ < 4 ? 1 : 2) void prefill_tiles_kernel(PrefillArgs args) {
  attend_items<DH, NWQ, MODE>(args);
}

template <int DH, int NWQ, Mode MODE>
int launch(const PrefillArgs& a, int64_t rows, hipStream_t st) {
  static std::atomic<int64_t> blocks{0};
  return launch_items(prefill_tiles_kernel<DH, NWQ, MODE>, NWQ, blocks, "prefill_tiles_kernel", a, rows, st);
}

template <int DH, Mode MODE>
int launch_waves(const PrefillArgs& a, int64_t rows, int nwq, hipStream_t st) {
  if (nwq == 4) return launch<DH, 4, MODE>(a, rows, st);
  if (nwq == 2) return launch<DH, 2, MODE>(a, rows, st);
  return launch<DH, 1, MODE>(a, rows, st);
}

template <int DH>
int launch_mode(const PrefillArgs& a, int64_t rows, int nwq, hipStream_t st) {
  if (a.full) return launch_waves<DH, Mode::Full>(a, rows, nwq, st);
  return a.K ? launch_waves<DH, Mode::Rows>(a, rows, nwq, st) : launch_waves<DH, Mode::Paged>(a, rows, nwq, st);
}

}  // namespace

int prefill_tiles_launch(const PrefillArgs& a, int64_t rows, int Dh, int nwq, hipStream_t st) {
  return Dh == 128 ? launch_mode<128>(a, rows, nwq, st) : launch_mode<64>(a, rows, nwq, st);
}

}  // namespace dllava
