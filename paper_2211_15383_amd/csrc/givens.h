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

// One wavefront: R^-1 g over the first k <= K columns, entry c in lane c (lanes from k on hold
// nothing), R the rotated Hessenberg matrix (column c at H + c ld), row by row from the last, each
// row's terms subtracted in the order of the columns; zero pivots give zero coefficients.
// Lane c has row c: t[l] holds R[c][l] and, once y_l is known (one broadcast a row), the term
// R[c][l] y_l; a row's subtractions are a chain in registers.  (With the terms in column lanes each
// took four readlanes, 28 clocks for two: 1270 clocks a row at k = 24.  Parts are selected one by
// one: as a whole the compiler selects between copies in scratch memory.)
template <int K>
__device__ __forceinline__ c128 givens_backsub(const c128* H, int ld, const c128* g, int k) {
  const int c = threadIdx.x & 63, row = c < k ? c : 0;
  c128 mine = g[row], t[K];
#pragma unroll
  for (int l = 0; l < K; ++l) t[l] = H[min(l, k - 1) * ld + row];
  const c128 hd = H[row * ld + row];
  const double dd = fma(hd.x, hd.x, hd.y * hd.y);
#pragma unroll
  for (int i = K - 1; i >= 0; --i) {  // rows from k on leave no term
    c128 acc = mine;
#pragma unroll
    for (int l = i + 1; l < K; ++l) acc = acc - t[l];
    const double nx = fma(acc.x, hd.x, acc.y * hd.y) / dd, ny = fma(acc.y, hd.x, -(acc.x * hd.y)) / dd;
    c128 y;
    y.x = dd > 0.0 ? nx : 0.0;
    y.y = dd > 0.0 ? ny : 0.0;
    mine.x = c == i ? y.x : mine.x;
    mine.y = c == i ? y.y : mine.y;
    const c128 term = cprod<false>(t[i], lane_value(y, i));
    t[i].x = i < k ? term.x : 0.0;
    t[i].y = i < k ? term.y : 0.0;
  }
  return mine;
}

// The same for any k <= 64 with the terms in the place of R (LDS), for a kernel that lacks the
// registers.
__device__ __forceinline__ c128 givens_backsub_lds(c128* H, int ld, const c128* g, int k) {
  const int c = threadIdx.x & 63, row = c < k ? c : 0;
  c128* hr = H + row;
  c128 mine = g[row];
  const c128 hd = hr[row * ld];
  const double dd = fma(hd.x, hd.x, hd.y * hd.y);
  for (int i = k - 1; i >= 0; --i) {
    const c128 h = hr[i * ld];
    c128 acc = mine;
    int l = i + 1;
    for (; l + 4 <= k; l += 4) {
      const c128 t0 = hr[l * ld], t1 = hr[(l + 1) * ld], t2 = hr[(l + 2) * ld], t3 = hr[(l + 3) * ld];
      acc = (((acc - t0) - t1) - t2) - t3;
    }
    for (; l < k; ++l) acc = acc - hr[l * ld];
    const double nx = fma(acc.x, hd.x, acc.y * hd.y) / dd, ny = fma(acc.y, hd.x, -(acc.x * hd.y)) / dd;
    c128 y;
    y.x = dd > 0.0 ? nx : 0.0;
    y.y = dd > 0.0 ? ny : 0.0;
    mine.x = c == i ? y.x : mine.x;
    mine.y = c == i ? y.y : mine.y;
    if (c < i) hr[i * ld] = cprod<false>(h, lane_value(y, i));
  }
  return mine;
}
