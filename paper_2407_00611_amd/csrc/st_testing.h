/* Entry points for the library's own tests and tuning runs.  They are exported, but they are not part of the
 * interface a user programs against (the public header does not declare them) and may change at any time. */
#pragma once

#include "../../include/startrail.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Sets one launcher switch for the rest of the process (not thread safe against running launches):
 *   "fwd_fast", "dq_fast", "dkv_fast"   0 keeps that pass entirely in the general kernels
 *   "dkv_queue"                         0 gives every dK/dV key tile a workgroup of its own
 *   "one_walk"                          0 keeps every ring backward in its two passes, 2 takes the one walk wherever it can
 *   "one_heads" (0 .. 8)                KV heads of a batch of the one walk, where they divide the heads (0: as planned)
 *   "one_polls" (1 ..)                  polls after which a wait of the one walk gives up (then every gradient is NaN)
 *   "fwd_wq" (32 | 64), "fwd_pipe"      variant of the general forward kernel
 *   "fwd_gap" (0 .. 64)                 log2 units a block maximum may exceed the lazy exponent reference by
 * Returns 0, or 1 for an unknown name or a value out of range (nothing changes then). */
int st_testing_set(const char* name, double value);

/* How a ring backward over the listed chunks would be split, without launching anything (host only): st_ring_bwd(_last) with a
 * workspace of so many bytes, or st_ring_bwd_noalloc (workspace_bytes < 0); mode -1: st_attn_block_bwd of each.  Writes 12 values per launch to out (host): chunks;
 * dQ: most shares of a query tile, shares of a head where the tiles differ, first shares that add themselves, shares per tile
 * (4 words); dK/dV: blocks per share, shares (all gradients in one walk: KV heads of a batch, negative); both passes in one launch; bytes of partial sums.  Returns the number of values,
 * or -1 if max_out are too few or the descriptor has no kernel. */
int st_testing_bwd_plan(const st_ring_desc* desc, const int32_t* order, int32_t n_visit, int32_t mode, int32_t assign,
                        int64_t workspace_bytes, int64_t* out, int32_t max_out);

/* Compute units and XCDs of the current device as the launchers see them; returns 0 if known. */
int st_testing_device(int* cus, int* xcds);

#ifdef __cplusplus
}
#endif
