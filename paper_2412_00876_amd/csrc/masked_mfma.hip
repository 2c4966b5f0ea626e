// Matrix-core attention of the training form, bfloat16 (Eq. 7 of the paper: the keep mask inside the softmax, over the full
// token set).  The kernel's body and what bounds it: attn_tiles.h.
#include "attn_tiles.h"

namespace dllava {

namespace {

template <int DH, Mode MODE>
__global__ __launch_bounds__(4 * kWave, 2) void masked_mfma_kernel(PrefillArgs args) {
  attend_items<DH, 4, MODE>(args);
}
// 104 vector and 64 accumulation registers: three waves per SIMD instead of two (16x32 sequences x heads of 320 rows 53 -> 40 us together
// with the mask of a tile as one word of bits per lane)
template <>
__global__ __launch_bounds__(4 * kWave, 2) __attribute__((amdgpu_num_vgpr(104))) void masked_mfma_kernel<64, Mode::Masked>(PrefillArgs args) {
  attend_items<64, 4, Mode::Masked>(args);
}
template <>
__global__ __launch_bounds__(4 * kWave, 2) __attribute__((amdgpu_num_vgpr(104))) void masked_mfma_kernel<64, Mode::Words>(PrefillArgs args) {
  attend_items<64, 4, Mode::Words>(args);
}

// Items of 128 rows whatever the size of the launch: over means of 32..768 rows and 1x8..64x40 sequences x heads the call takes
// 0.64..0.89 of what it took on the kernel before (which was level with smaller items at every size).  (Measured before the visible
// keys came from a list.)
template <int DH, Mode MODE>
int launch(const PrefillArgs& a, int64_t rows, hipStream_t st) {
  static std::atomic<int64_t> blocks{0};
  return launch_items(masked_mfma_kernel<DH, MODE>, 4, blocks, "masked_mfma_kernel", a, rows, st);
}

}  // namespace

// returns 1 if the shape is not handled here
int masked_mfma_launch(const PrefillArgs& a, int64_t rows, int Dh, hipStream_t st) {
  const bool list = a.mask_slots > 0;
  if (Dh == 128) return list ? launch<128, Mode::Masked>(a, rows, st) : launch<128, Mode::Words>(a, rows, st);
  if (Dh == 64) return list ? launch<64, Mode::Masked>(a, rows, st) : launch<64, Mode::Words>(a, rows, st);
  return 1;
}

}  // namespace dllava
