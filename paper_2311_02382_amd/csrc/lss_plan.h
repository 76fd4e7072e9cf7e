/*
 * lss_plan.h -- which kernels a call launches, for the tests that are about one of them; not part of the library's
 * product interface (include/lss_attn.h).  Host only: nothing is launched.
 *
 *   lss_plan_fwd  forward with a workspace of lss_workspace_bytes():  plan[0] blocks of 32 query rows of a workgroup,
 *                 plan[1] groups of wavefronts that have a part of its keys each, plan[2] key splits
 *   lss_plan_bwd  backward; `over_out`: a gradient overlaps the forward's output.  plan[0] key splits of dQ, plan[1] groups,
 *                 plan[2] all three gradients in one pass, plan[3] no preprocess launch, plan[4] dK/dV workgroups for at most
 *                 64 rows, plan[5] wavefronts of 16 rows
 *
 *   lss_plan_linear   op 0 lss_linear_fwd, 1 lss_linear_bwd_input, 2 lss_linear_bwd_weight (fused forms take the same tiles).  plan[0] tile (GemmTile
 *                     of lss_gemm_plan.h), plan[1] chunks of rows, plan[2] groups of wavefronts that share a contraction, plan[3] slots of their rings
 *   lss_plan_project  op 0 lss_project_qkv, 1 lss_project_bwd: plan[0] tile, plan[1] groups, plan[2] slots;  op 2 lss_project_bwd_weight: plan[0] tile and
 *                     plan[1] chunks of rows per batch entry of dW_q, plan[2] and plan[3] of dW_kv, plan[4] groups and plan[5] slots of dW_q, plan[6] and
 *                     plan[7] of dW_kv.  `rows_valid` is not looked at for op 0; at least one row of all kinds
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
int lss_plan_linear(int op, int64_t rows, int64_t K, int64_t N, int *plan);
int lss_plan_project(int op, int64_t l_s, int64_t l_x, int64_t rows_valid, int64_t B, int64_t H, int64_t d, int *plan);

#ifdef __cplusplus
}
#endif
#endif /* LSS_PLAN_H */
