// Arguments of the prefill-attention kernels.
#pragma once

#include "common.h"

namespace dllava {

struct PrefillArgs {
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  const int32_t* off;
  int32_t B, H;
  float scale_log2;
  // keys/values come from the paged cache when K == nullptr
  const void* pages;
  const int32_t* block_table;
  int32_t max_pages;
  // 0: causal (query i sees keys 0..i of its sequence); 1: every query sees all keys of its sequence
  int32_t full;
  // Key masks (Eq. 7), or null: bit i of word t of sequence b says whether key 32t + i may be seen by LATER queries
  // (a query always sees itself); the words of sequence b start at key_words[off[b] / 32 + b].  masked_mfma_launch only.
  const uint32_t* key_words;
  // mask_slots > 0: behind the words, mask_slots words on, as many counts, one for each word: for word 4i of a sequence (where the
  // queries of an item of 128 begin) the visible keys of the sequence in front of it, for the word before that, 4i - 1, the words that
  // are not zero in front of 4i.  Behind those the visible keys as a list: entry off[b] + 32 b + r is where the row of sequence b's
  // visible key r starts, in bytes (mod 2^32) from the row of its key 0.
  int32_t mask_slots;
};

// A value of DLLAVA_LAUNCH_PREFILL_WAVES: 1, 2 or 4 waves, or 0; plus 16 (the kernel for long sequences) or 32 (the one for short
// ones), or neither.  Any other value counts as 0.
struct ForcedForm {
  int waves;        // 0: automatic
  bool tiles, few;  // long, short; neither: automatic
};
constexpr ForcedForm forced_form(int v) {
  const int waves = v & 15, kernel = v & ~15;
  if ((waves != 0 && waves != 1 && waves != 2 && waves != 4) || (kernel != 0 && kernel != 16 && kernel != 32)) return {0, false, false};
  return {waves, kernel == 16, kernel == 32};
}

// matrix-core path (prefill_mfma.hip); returns 1 if it does not handle the shape
int prefill_mfma_launch(const PrefillArgs& a, int64_t rows, int Dh, hipStream_t st);
// its software-pipelined kernel (prefill_tiles.hip), blocks of nwq waves; Dh 64 or 128; 1 if the launch would be too large
int prefill_tiles_launch(const PrefillArgs& a, int64_t rows, int Dh, int nwq, hipStream_t st);
// the causal form over rows with key masks (masked_mfma.hip); returns 1 if it does not handle the shape
int masked_mfma_launch(const PrefillArgs& a, int64_t rows, int Dh, hipStream_t st);

}  // namespace dllava
