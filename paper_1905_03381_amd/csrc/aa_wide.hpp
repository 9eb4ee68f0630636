// Host-side launch interface of the passes over dense rows the aligned register layouts do not
// take: the block-per-row pass over wide ones, the any-address rows of k_step_pass below that.
#pragma once

#include "aa_dense.hpp"

namespace aa {

constexpr int kWideMinD = 1025;  // (narrower rows, which leave most of a block's threads without a column, go a row per wave)
constexpr int kAnyMinD = 4;      // one piece of four floats
constexpr int kWideMaxD = 8192;  // columns the registers of one block hold
constexpr int kWideBlocks = 256;  // one per compute unit

// Whether the scoring pass reads a matrix of that size with plain loads.  A matrix that stays in the
// 256 MB memory-side cache from one pass to the next loses by non-temporal ones, unless it is so small
// that the rest of the cache takes them too.  Every row scored again and again, plain / non-temporal
// loads (the general kernel in brackets): 20,000 x 1027 (82 MB) 16.3 / 17.4 us (16.6), 60,000 x 1027
// (246 MB) 39.7 / 47.4 (39.8), 30,000 x 2047 36.4 / 38.6 (35.5), 20,000 x 3000 35.0 / 36.6 (35.2), but 9000 x 2047
// (74 MB) 13.3 / 12.4 (13.3) and 4096 x 4137 (68 MB) 11.7 / 10.8 (12.8); rows not seen before, out of 3 GB:
// 20,000 x 1367 23.6 / 21.5 (24.2), 20,000 x 3000 44.4 / 39.8 (45.7).
inline bool wide_plain_loads(size_t matrix_bytes) {
  return matrix_bytes > ((size_t)76 << 20) && matrix_bytes <= (size_t)256 << 20;
}

// True if these passes take the rows; the aligned register layouts come first.
bool wide_rows_ok(const aa_features *F);

// Padded width (floats) of one gradient partial.
int32_t wide_d_pad(int32_t d);

// Passes that update both vectors leave a block's sums of the columns from this one on in doubles.
constexpr int kWideFp32Cols = 4096;

// Floats of a block's sums of one vector: the padded row, the doubles counting twice.
int32_t wide_part_row(int32_t d, int nvec);

int32_t wide_pass_blocks(int32_t d, int32_t count);

hipError_t launch_wide_pass(const PassArgs &a, int mode, int32_t nblk, hipStream_t stream,
                            hipEvent_t started = nullptr, hipEvent_t stopped = nullptr);

}  // namespace aa
