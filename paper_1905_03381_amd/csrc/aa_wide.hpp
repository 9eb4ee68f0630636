// Host-side launch interface of the passes over dense rows the aligned register layouts do not
// take: the block-per-row pass over wide ones, the any-address rows of k_step_pass below that.
#pragma once

#include "aa_dense.hpp"

namespace aa {

constexpr int kWideMinD = 1025;  // (narrower rows, which leave most of a block's threads without a column, go a row per wave)
constexpr int kAnyMinD = 4;      // one piece of four floats
constexpr int kWideMaxD = 8192;  // columns the registers of one block hold
constexpr int kWideBlocks = 256;  // one per compute unit

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
