/*
 * qmoe_hooks.h -- measurement hooks of libqmoe.so.  NOT part of the product ABI (qmoe.h):
 * they exist so that a benchmark or a profiler run can time one kernel of a layer call on a
 * workspace that a full call has filled, or switch one staging decision off.  Process-wide,
 * not thread-safe against running calls; nothing in the product path sets them.
 */
#ifndef QMOE_HOOKS_H
#define QMOE_HOOKS_H

#include "qmoe.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Keys:
 *  "phases"    bit mask of the kernels qmoe_moe_layer_forward / qmoe_bf16_layer_forward enqueue:
 *              1 dispatch, 2 / 4 scalar kernel of the first / second product, 8 / 16
 *              matrix-core kernel of the first / second product (in calls that bring the activations
 *              in blocks: 8 with the copy, into y, and 16 clears the rows of tokens without an
 *              expert); 0 = all (the default)
 *  "stage_out" -1 = the products write their results straight to global memory instead of
 *              staging a block's results in LDS; 0 = default
 *  "rows"      1 = layer calls and single matrices use the kernel with several lanes per row
 *              wherever it can run, -1 = never, 0 = the planner's choice (the default)
 *  "encode_rows" n = the device encoder takes at most n rows (in whole groups of its wavefronts) in a round of its three
 *              kernels, as it does by itself from 2^31 values on; 0 = default
 * Unknown key: QMOE_E_INVALID_ARG.
 */
qmoe_status qmoe_hook_set(const char *key, int value);

/*
 * 1 if a layer call of this size gives its experts with few tokens to the kernel with several lanes per
 * row, 0 if to the one with a row range per lane (also on error): the name of the kernel that a profile
 * shows (widths whose activations leave room for tiles of four tokens).  format: QMOE_FORMAT_* bits.
 */
int qmoe_hook_several_lanes(const qmoe_dict *d, int format, int n_experts, int d_model, int d_ff, int n_tokens);

/*
 * How the kernel with several lanes per row cuts a launch into one share per workgroup, computed on the host (no GPU needed):
 * items[0], [1], [2] token tiles of three or four, two, one tokens, in this order, of matrices of `rows` rows; tiles_at_once: 1, or
 * 2 where the activations of two tiles fit the LDS.  Share b goes from row out[4 b + 1] of item out[4 b] to row out[4 b + 3] of
 * item out[4 b + 2], and is empty if that is a lower item.  out: int[4 * groups].
 */
qmoe_status qmoe_hook_rows_shares(int rows, const int items[3], int tiles_at_once, int groups, int *out);

#ifdef __cplusplus
}
#endif
#endif /* QMOE_HOOKS_H */
