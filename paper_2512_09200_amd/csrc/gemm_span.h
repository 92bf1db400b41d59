// Which operands the GEMMs' buffer loads can address (host rules, plain C++).
#pragma once
#include <stdint.h>

namespace lat {

// Bytes from a bf16 operand's first element to the end of its last one: R rows
// (or columns) of K, K-contiguous (rows of ld) or not (mn).
inline int64_t operand_span(int64_t ld, int R, int K, bool mn) {
  if (R <= 0 || K <= 0) return 0;
  return mn ? ((int64_t)(K - 1) * ld + (R + 7) / 8 * 8) * 2 : ((int64_t)(R - 1) * ld + (K + 7) / 8 * 8) * 2;
}

// k that the last loads of the loops may address past the range: the rest of
// the last step of 64, and the few-tile kernel's loads three steps ahead.
constexpr int BUF_AHEAD = 64, BUF_AHEAD_DMA = 320;

// Within 2 GiB counting the k addressed past the range: their byte offsets must
// stay below 2^32, out of the resource's range, so that they read zero rather
// than wrap back into it.
inline bool operand_in_buffer(int64_t ld, int R, int K, bool mn, int ahead) {
  return operand_span(ld, R, K, mn) + ahead * (mn ? ld : 1) * 2 < (int64_t)1 << 31;
}

}  // namespace lat
