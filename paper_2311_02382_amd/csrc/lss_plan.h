/*
 * lss_plan.h -- which kernels an attention call launches, for the tests that are about one of them; not part of the library's
 * product interface (include/lss_attn.h).  Host only: nothing is launched.
 *
 *   lss_plan_fwd  forward with a workspace of lss_workspace_bytes():  plan[0] blocks of 32 query rows of a workgroup,
 *                 plan[1] groups of wavefronts that have a part of its keys each, plan[2] key splits
 *   lss_plan_bwd  backward; `over_out`: a gradient overlaps the forward's output.  plan[0] key splits of dQ, plan[1] groups,
 *                 plan[2] all three gradients in one pass, plan[3] no preprocess launch, plan[4] dK/dV workgroups for at most
 *                 64 rows, plan[5] wavefronts of 16 rows
 *
 * Returns LSS_OK or a negative lss_status.
 */
#ifndef LSS_PLAN_H
#define LSS_PLAN_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

int lss_plan_fwd(int64_t seg_offset, int64_t l_s, int64_t l_x, int64_t B, int64_t H, int64_t d, int causal, int with_dropout,
                 int elem_bytes, int *plan);
int lss_plan_bwd(int64_t seg_offset, int64_t l_s, int64_t l_x, int64_t B, int64_t H, int64_t d, int causal, int with_dropout,
                 int elem_bytes, int over_out, int *plan);

#ifdef __cplusplus
}
#endif
#endif /* LSS_PLAN_H */
