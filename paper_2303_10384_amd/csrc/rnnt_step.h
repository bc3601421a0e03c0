// The loss in two calls, for the package's autograd wrapper (not part of the public C-ABI):
// the losses and the row records of the gradient first, the gradient when the upstream
// gradient is known.  Arguments as in rnnt_loss (include/rnnt_mi355x.h); a given workspace is all they use.
#pragma once

#include "rnnt_mi355x.h"

#ifdef __cplusplus
extern "C" {
#endif

// Bytes of workspace of rnnt_step_forward (0 for an invalid shape).
size_t rnnt_step_workspace_bytes(rnnt_shape_t shape);

// Columns of 64 units of the scaled sweep that the loss takes lattices of up to U_max units through, 0 for
// the log2 sweep (for tests of what a shape reaches).
int32_t rnnt_scaled_sweep_columns(int32_t U_max);

// Losses, and in rows_out the row records: 16 bytes for each of the B * T_max * (U_max+1)
// logits rows, 16-byte aligned.  workspace: 256-byte aligned, free again after the call's work, or NULL (the
// library takes one as in rnnt_loss).
rnnt_status_t rnnt_step_forward(const void* logits, rnnt_shape_t shape, const int32_t* labels,
                                const int32_t* logit_lens, const int32_t* label_lens, int32_t blank,
                                rnnt_variant_t variant, float* loss_out, void* rows_out, void* workspace,
                                size_t workspace_bytes, hipStream_t stream);

// The gradient of the losses from the same logits and the rows of rnnt_step_forward, in the
// logits' type.  scale: NULL, or device float32, one value (scale_per_utterance = 0) or B
// values; every element of utterance b, padding included, is multiplied by scale / divisor in
// float32 before it is stored.
rnnt_status_t rnnt_step_gradient(const void* logits, rnnt_shape_t shape, int32_t blank, const void* rows,
                                 const float* scale, int32_t scale_per_utterance, float divisor, void* grad_out,
                                 hipStream_t stream);

#ifdef __cplusplus
}
#endif
