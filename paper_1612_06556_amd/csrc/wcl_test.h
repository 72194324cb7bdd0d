/*
 * wcl_test.h -- entry points of libwcl.so for its tests; not part of the API
 * (include/wcl.h), no binding.
 */
#ifndef WCL_TEST_H
#define WCL_TEST_H

#include "../../include/wcl.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The hopping kernel in the launch shape set in the context (wcl_set_tuning,
 * wcl_set_hop_staging, wcl_set_hop_tiles, wcl_set_batch_tuning), on canonical
 * complex128 [nrhs][V][4][3] device buffers, with links and clover in
 * link_prec and vectors in vec_prec (64, 32 or 16):
 *   WCL_OP_HOP    out = H in, one launch per parity as wcl_bench_hop times it
 *                 (vec_prec 32)
 *   WCL_OP_SCHUR  out_e = Dhat in_e, out_o = 0, by the solver's two launches on
 *                 lattices of any size; dots 1 or 2: with the inner products
 *                 of the solver's iteration in the second (their sums unused)
 *   WCL_OP_D      out = D in, by the two launches of the solver's residuals (64)
 * Allocates its fields for the call and synchronises the stream. */
int wclt_hop(wcl_ctx *ctx, int op, const double *in_dev, double *out_dev, int nrhs, int link_prec, int vec_prec, int dots);

#ifdef __cplusplus
}
#endif
#endif
