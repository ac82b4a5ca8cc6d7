/*
 * loopserve_test_hooks.h -- entry points of libloopserve that exist for its tests only.  They know
 * internals (workspace layout, kernel wait bounds) and are not part of the product interface.
 */
#ifndef LOOPSERVE_TEST_HOOKS_H
#define LOOPSERVE_TEST_HOOKS_H

#include "loopserve.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Copies the retention score [B,Hkv,len] fp32 (column sums of the last n_obs rows, summed over each
 * KV group, Sec. 5.2) that the most recent ls_kv_compress call on this context left in the workspace
 * to `dst_device`.  `shape` must be the shape of that call.
 */
int ls_debug_copy_compress_score(ls_ctx* ctx, const ls_shape* shape, float* dst_device, void* hip_stream);

/*
 * Bound (number of polls) of every wait between the waves of the greedy-loop kernel of ls_select on
 * this context; negative restores the default.  With a bound of 0 a wave that has to wait gives up at
 * once, every wave still leaves the kernel normally, and the heads concerned take the documented
 * LS_STAT_WALK_TIMEOUT path: this is how the tests reach that path from the host.
 */
int ls_debug_set_walk_spin_limit(ls_ctx* ctx, int32_t limit);

/*
 * Sets every counter through which workgroups of one launch find out which of them is the last to `value`
 * (zero between calls).  The tests use it to see that calls recover from counters that are off.
 */
int ls_debug_set_counters(ls_ctx* ctx, int32_t value, void* hip_stream);

/*
 * Sets every word of the context's workspace to `value`: what a call finds there is whatever an earlier one left, and the tests see that no
 * result depends on it.
 */
int ls_debug_fill_workspace(ls_ctx* ctx, int32_t value, void* hip_stream);

/*
 * Copies to the host how the most recent ls_sparse_prefill call on this context shared its items among the XCDs, as its kernels
 * left it in the workspace: its work queues, or in a call that needs none the items that begin on each XCD's workgroups (an item is one
 * block of 128 query rows of one head).  host_queue holds 8 arrays of B * Hq * nqb words, (batch * Hq + head) << 16 | row block, of
 * which the first host_qlen[x] are valid; *nqb_out receives the number of row blocks per head, *cuts_out how many cuts go through items.
 * `shape` must be that call's shape.  Waits for the stream.  The tests use it to check that every item is there exactly once, and
 * that items are cut where the workspace has room for their parts.
 */
int ls_debug_copy_prefill_queues(ls_ctx* ctx, const ls_shape* shape, uint32_t* host_queue, int32_t* host_qlen,
                                 int32_t* nqb_out, int32_t* cuts_out, void* hip_stream);

/*
 * How far the most recent call on this context, an ls_select of this shape that was not asked for the accounted mass, put its lists in order, as its kernels
 * left it in the workspace: *ranges receives the ranges of each list (0: a call of this shape and workspace leaves none out), host_left [2][B * Hq] how many
 * of them were left out to the end (diagonals, then columns), host_again [B * Hq] how many had been, of heads that were then walked again with everything in order (else 0).  Waits for the stream.
 */
int ls_debug_copy_select_order(ls_ctx* ctx, const ls_shape* shape, int32_t* host_left, int32_t* host_again, int32_t* ranges, void* hip_stream);

/* 1: ls_sparse_prefill shares the work of such a turn out in pieces, 0: by work queues, if the workspace has room for the parts; without a GPU. */
int ls_debug_prefill_in_pieces(const ls_shape* shape);

/*
 * Which of the scoring passes' kernels a call of this shape takes and how it cuts the keys, without a GPU.  `mode`: 0 ls_score of the newest
 * rows (w <= 128), 1 ls_score otherwise, 2 ls_kv_compress, 3 ls_score_window; `positions`: with explicit positions.  route[0]: ranges of keys of the statistics pass (0: a workgroup per
 * 128 keys), [1] chunks of 32 rows that a workgroup of it takes at most, [2] workgroups that share a KV head's query heads, [3] row statistics are merged by the second pass,
 * [4] key blocks join their results themselves, [5] the retention's second pass keeps its rows and streams the keys; mode 1, with the
 * workspace that ls_workspace_bytes states: [6] KV heads and [7] rows of a band of the window matrix, [8] workgroups of the first that share a KV head's query heads.  begins (may be NULL): of route[0] + 1
 * words, the key at which each range begins, and n.
 */
int ls_debug_score_route(const ls_shape* shape, int32_t mode, int32_t positions, int32_t route[9], int64_t* begins);

#ifdef __cplusplus
}
#endif
#endif /* LOOPSERVE_TEST_HOOKS_H */
