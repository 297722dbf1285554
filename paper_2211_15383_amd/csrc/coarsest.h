// Whole fixed-count GMRES of small coarsest levels in one launch (coarsest.hip).
#pragma once

#include "common.h"

// Whether coarsest_small runs the m-step GMRES of level L, with a deflation of k vectors (0:
// none), in precision R.
template <typename R>
bool coarsest_small_ok(const Level& L, int m, int k);
// Bytes of device scratch it needs for nrhs right-hand sides (0 when the basis fits in LDS).
template <typename R>
size_t coarsest_small_scratch(const Level& L, int m, int k, int nrhs);
// x = e0 + GMRES_m(D, r) with r = b - W W^H b and e0 = X Lambda^-1 W^H b for the deflation D
// of this level (r = b, e0 = 0 without); b, x: [nrhs][n].
template <typename R>
void coarsest_small(dmlmc_ctx* ctx, const Level& L, const dmlmc_defl* D, const Cx<R>* b, Cx<R>* x, int nrhs, int m,
                    void* scratch);
