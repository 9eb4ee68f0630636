// Host-side launch interface of the epochs over small pools.
#pragma once

#include "aa_common.hpp"

namespace aa {

struct SmallEpochArgs {
  const float *x;
  int64_t ld;
  int32_t d, d4;
  const float *y;
  const int32_t *perm;    // pool t is perm[t * P : min((t + 1) * P, n_perm)]
  int64_t n_perm;
  int32_t P, steps;       // steps of this launch
  float *w, *phi, *bias;  // phi and bias NULL for hard thresholds; bias may be NULL
  const float *T;
  float gamma, one_minus_gamma;
  uint32_t k0, k1;        // Philox key
  uint64_t step;          // Philox step of the first pool
  float lambda, lr, lr_a, l2_a;
  int32_t *t_upd;
  int32_t *kept_hist;     // [steps] or NULL
  // the batch of each step; pool t's ids start at t * ids_stride, its losses at t * loss_stride
  // (0: every step writes the same place)
  int32_t *ids, *kept_pos;
  float *loss, *prob;
  uint8_t *flags;
  int64_t ids_stride, loss_stride;
  // what the blocks of a team tell each other, small_epoch_words_bytes() bytes (NULL: no team), and a control word of the
  // workspace with which tests end a team: 2: the gate is shut from the start; 4 (t + 1) + b: block b leaves in step t, as if
  // the others' words had not come; anything else, as the zero that preparing a workspace leaves there, does nothing
  uint64_t *words;
  const int32_t *ends;
};

constexpr int kSmallEpochSteps = 1024;  // steps of one launch at most

// True if pools of P rows of d floats (16-byte aligned, d % 4 == 0) fit the registers of a block.
bool small_epoch_ok(int32_t d, int64_t ld, int32_t P);

size_t small_epoch_words_bytes();

hipError_t launch_small_epoch(const SmallEpochArgs &a, bool hard, hipStream_t stream);

}  // namespace aa
