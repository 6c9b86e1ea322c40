/* lbm_rollout.h -- entry points that the package calls besides the C ABI of
 * lbm.h: whole pieces of a rollout's schedule in fewer passes over memory than
 * its single calls take, and which kernels a context's steps take.  The
 * binding's own; a user's program has everything it needs in lbm.h. */
#ifndef LBM_ROLLOUT_H
#define LBM_ROLLOUT_H

#include "lbm.h"

#ifdef __cplusplus
extern "C" {
#endif

/* n >= 1 steps of lbm_step_state from src_state (NULL: the context's current
 * state) into dst_state (NULL: the context's current state), two to a pass
 * where lbm_step would take them so; bitwise n single ones.  Snapshots as
 * there.  The first pass reads src_state and the last one writes dst_state;
 * those in between use the context's population buffers, so with dst_state the
 * context's own state is an earlier one of the n afterwards (or unchanged, if
 * one pass was enough).  lbm_bc needs a propagate first, as after
 * lbm_set_state. */
lbm_status lbm_advance_state(lbm_ctx* ctx, void* src_state, void* dst_state, int64_t n);

/* How lbm_step takes two steps in one pass over memory in this context. */
typedef enum {
    LBM_TWO_STEP_NONE = 0,      /* it does not: single steps */
    LBM_TWO_STEP_TILE_8X8 = 1,  /* tiles of that many columns and rows */
    LBM_TWO_STEP_TILE_8X16 = 2,
    LBM_TWO_STEP_TILE_16X16 = 3,
    LBM_TWO_STEP_MARCH = 4      /* a march along x */
} lbm_two_step;
lbm_two_step lbm_two_step_form(const lbm_ctx* ctx);

#ifdef __cplusplus
}
#endif
#endif
