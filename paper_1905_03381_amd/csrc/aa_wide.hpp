// Host-side launch interface of the block-per-row pass over wide dense rows.
#pragma once

#include "aa_dense.hpp"

namespace aa {

constexpr int kWideMinD = 1025;  // (narrower rows leave most of a block's threads without a column)
constexpr int kWideMaxD = 8192;  // columns the registers of one block hold
constexpr int kWideBlocks = 256;  // one per compute unit

// True if k_wide_pass takes these rows; the register-resident kernels come first.
bool wide_rows_ok(const aa_features *F);

// Padded width (floats) of one gradient partial.
int32_t wide_d_pad(int32_t d);

int32_t wide_pass_blocks(int32_t count);

hipError_t launch_wide_pass(const PassArgs &a, int mode, int32_t nblk, hipStream_t stream,
                            hipEvent_t started = nullptr, hipEvent_t stopped = nullptr);

}  // namespace aa
