/*
 * Calls of na2d.h and na1d.h with the bias gradient in the problem's dtype instead of fp32: the fp32 sums are rounded once, to nearest
 * even, by the kernel that stores them.  Everything else is as in the calls of the same names without "_typed".
 */
#ifndef NA_TYPED_H_
#define NA_TYPED_H_

#include "na1d.h"
#include "na2d.h"

#ifdef __cplusplus
extern "C" {
#endif

int na2d_qk_bwd_rpb_typed(const na2d_problem *p, const void *ds, void *d_rpb, void *workspace, size_t workspace_bytes, void *stream);
int na2d_fused_bwd_typed(const na2d_problem *p, const void *q, const void *k, const void *v, const void *rpb,
                         float scale, const float *lse, const void *dout, void *dq, void *dk, void *dv, void *d_rpb,
                         void *workspace, size_t workspace_bytes, void *stream);
int na2d_direct_bwd_typed(const na2d_problem *p, const void *q, const void *k, const void *v, const void *rpb,
                          float scale, const float *lse, const void *dout, void *dq, void *dk, void *dv, void *d_rpb,
                          void *workspace, size_t workspace_bytes, void *stream);
int na1d_fused_bwd_typed(const na1d_problem *p, const void *q, const void *k, const void *v, const void *rpb, float scale,
                         const float *lse, const void *dout, void *dq, void *dk, void *dv, void *d_rpb, void *workspace,
                         size_t workspace_bytes, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* NA_TYPED_H_ */
