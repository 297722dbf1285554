// Whole fixed-count GMRES of small coarsest levels in one launch (coarsest.hip).
#pragma once

#include "common.h"

// Whether coarsest_small runs the m-step GMRES of level L on nrhs right-hand sides in precision R.
template <typename R>
bool coarsest_small_ok(const Level& L, int m, int nrhs);
// Whether it takes in a deflation of k vectors too; small_deflate comes before it otherwise.
template <typename R>
bool small_deflates_inside(const Level& L, int k);
// r = b - W W^H b and e0 = X Lambda^-1 W^H b for the deflation D of a level of at most
// SMALL_LEVEL_N entries; b, r, e0: [nrhs][n], c: scratch of 2 k nrhs entries.
template <typename R>
void small_deflate(dmlmc_ctx* ctx, const Level& L, const dmlmc_defl* D, const Cx<R>* b, int nrhs, c128* c, Cx<R>* r,
                   c128* e0);
// Bytes of device scratch coarsest_small needs for nrhs right-hand sides and k vectors deflated
// inside (0 when the basis fits in LDS).
template <typename R>
size_t coarsest_small_scratch(const Level& L, int m, int k, int nrhs);
// x = e0 + GMRES_m(D, r) with r and e0 as above for the deflation D of this level; without (D
// NULL) r = b, and e0 is the caller's (NULL: 0).  b, x: [nrhs][n].
template <typename R>
void coarsest_small(dmlmc_ctx* ctx, const Level& L, const dmlmc_defl* D, const Cx<R>* b, Cx<R>* x, int nrhs, int m,
                    void* scratch, c128* e0);
