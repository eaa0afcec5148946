// Which kernel a call runs: rules on sizes, formats and strides alone, in plain C++
// (no HIP), so that a CPU test can ask them for any shape.
#pragma once
#include <stdint.h>

namespace reqat {

// Format selector shared by the launchers (same values as the C ABI enum).
enum Fmt : int { kNV = 0, kMX = 1 };

// NVFP4 with a computed global scale: tensors of at most this many elements are small
// enough for every workgroup to read whole (from L2) for the maximum, so that codes and
// scale take one launch (kGLocal) instead of a pass and a fix-up.
// Dense rows are walked as one run of vectors: 384 KB.  One launch / two, us in a graph:
// 16 x 1536 3.3 / -, 33 x 2048 4.5 / 6.7, 64 x 1536 4.5 / 6.6, 16 x 8960 5.8 / 6.8, 10 x 18944
// 6.4 / 6.8; it grows by 0.6 to 0.3 us per 2^15 elements, the two launches hardly.
// Rows with a stride cost a division and a filter of non-finite values per vector in every
// workgroup: 16 x 4096 6.1 / -, 33 x 2048 7.8 / 6.8, 24 x 5120 9.5 / 6.8, 96 x 2048 12.8 / 6.9.
constexpr int64_t kLocalMaxElems = int64_t(3) << 16;
constexpr int64_t kLocalMaxElemsStrided = int64_t(1) << 16;

inline bool nv_one_launch(int64_t elems, bool dense) {
    return elems <= (dense ? kLocalMaxElems : kLocalMaxElemsStrided);
}

}  // namespace reqat
