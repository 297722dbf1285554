// The small dense pieces of a GMRES step, worked on by one wavefront with the data in LDS:
// Givens rotation of a Hessenberg column and the final back substitution.  The roundings
// (fused multiply-adds included) are fixed here, so every form of the step gives the same bits.
#pragma once

#include "common.h"

// a b with the first product of each part fused onto the second (IM_HX: which of the
// imaginary part's products is the fused one)
template <bool IM_HX>
__device__ __forceinline__ c128 cprod(c128 a, c128 b) {
  const double re = fma(a.x, b.x, -(a.y * b.y));
  return cmk(re, IM_HX ? fma(a.x, b.y, a.y * b.x) : fma(a.y, b.x, a.x * b.y));
}

// Applies rotations 0 .. j-1 (rc, rs) to column j of the Hessenberg matrix (entries 0 .. j,
// its subdiagonal entry beta >= 0 real), forms rotation j and takes g through it.  In every
// lane of the calling wavefront alike; col, rc, rs and g in LDS.
__device__ __forceinline__ void givens_column(c128* col, double beta, double* rc, c128* rs, c128* g, int j) {
  c128 a = col[0];
#pragma unroll 4
  for (int i = 0; i < j; ++i) {
    const c128 b = col[i + 1], s = rs[i];
    const double c = rc[i];
    const c128 sb = cprod<false>(s, b);
    col[i] = cmk(fma(a.x, c, sb.x), fma(a.y, c, sb.y));
    a = cmk(fma(c, b.x, -fma(a.x, s.x, a.y * s.y)), fma(c, b.y, -fma(a.y, s.x, -(a.x * s.y))));
  }
  const double aa = sqrt(fma(a.x, a.x, a.y * a.y));
  const double rho = sqrt(fma(beta, beta, aa * aa));
  double c = 1.0;
  c128 s = cmk(0.0, 0.0), diag = cmk(0.0, 0.0);
  if (rho != 0.0) {
    if (aa == 0.0) {
      c = 0.0;
      s = cmk(1.0, 0.0);
      diag = cmk(beta, 0.0);
    } else {
      const c128 ph = cmk(a.x / aa, a.y / aa);
      c = aa / rho;
      s = (beta / rho) * ph;
      diag = rho * ph;
    }
  }
  const c128 gj = g[j];
  __builtin_amdgcn_wave_barrier();
  col[j] = diag;
  rc[j] = c;
  rs[j] = s;
  g[j] = c * gj;
  g[j + 1] = cmk(-fma(s.x, gj.x, s.y * gj.y), -fma(s.x, gj.y, -(s.y * gj.x)));  // -conj(s) g_j
}

__device__ __forceinline__ c128 lane_value(c128 v, int lane) {
  return cmk(__hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v.x), lane),
                              __builtin_amdgcn_readlane(__double2loint(v.x), lane)),
             __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v.y), lane),
                              __builtin_amdgcn_readlane(__double2loint(v.y), lane)));
}

// One wavefront: g <- R^-1 g over the first k columns (k <= 60), R the rotated Hessenberg
// matrix (column c at H + c ld), row by row from the last, each row's terms subtracted in
// the order of the columns; zero pivots give zero coefficients.  Lane c holds g_c, then y_c.
__device__ __forceinline__ void givens_backsub(const c128* H, int ld, c128* g, int k) {
  const int c = threadIdx.x & 63;
  const c128* col = H + (c < k ? c : 0) * ld;
  c128 mine = g[c < k ? c : 0];
  c128 h = col[k - 1];
  for (int i = k - 1; i >= 0; --i) {
    const c128 hi = h;
    if (i > 0) h = col[i - 1];
    // lane l > i: R[i][l] y_l; zero beyond the last column, so that four at a time may overrun
    const c128 term = c < k ? cprod<false>(hi, mine) : cmk(0.0, 0.0);
    c128 acc = mine;
    for (int l = i + 1; l < k; l += 4) {
      const c128 t0 = lane_value(term, l), t1 = lane_value(term, l + 1), t2 = lane_value(term, l + 2),
                 t3 = lane_value(term, l + 3);
      acc = ((acc - t0) - t1) - t2;
      acc = acc - t3;
    }
    const double dd = fma(hi.x, hi.x, hi.y * hi.y);
    if (c == i)
      mine = dd > 0.0 ? cmk(fma(acc.x, hi.x, acc.y * hi.y) / dd, fma(acc.y, hi.x, -(acc.x * hi.y)) / dd)
                      : cmk(0.0, 0.0);
  }
  if (c < k) g[c] = mine;
}
