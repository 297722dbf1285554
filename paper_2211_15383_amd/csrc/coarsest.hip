// Fixed-count GMRES of a small coarsest level, every step of it in one launch.
//
// A V-cycle ends in m steps of GMRES on the coarsest operator (after the exact solve on the
// deflation space when one is attached).  As separate launches that is 3 or 4 launches a step
// and a dozen around them, 2 to 6 us each on vectors of a few KB: launch latency and idle
// CUs.  Here one workgroup owns one right-hand side: the Krylov vector, the operator's result,
// the Hessenberg matrix and (where it fits) the basis stay in LDS, and the operator's blocks
// are streamed from L2, which is what bounds a step (64 bytes per clock and CU).
//
//   * operator: a thread per row (column-major blocks, so that a wavefront's loads are
//     contiguous; the complex-FP32 d = 16 blocks, row-major for the matrix cores, have a
//     copy by column pairs on levels of this size).  In complex FP64 the contraction is split
//     over P threads where the rows alone would leave threads idle.  The short loops are
//     straight-line where the sizes allow it: a uniform branch for each load and product, and
//     the integer divisions of the site numbers, took longer than the products;
//   * Gram-Schmidt as in gram.hip: complex FP32 one pass on the unnormalised basis, complex
//     FP64 two passes on the normalised one; FP64 arithmetic;
//   * the last wavefront applies the Givens rotations to a step's Hessenberg column before it
//     joins the next step's operator, whose streaming hides them; one wavefront ends with the
//     back substitution.
//
// The complex-FP32 form performs the operations of the separate launches (the split Gram-Schmidt
// step, the coarse stencils, the coefficient kernels) in their order, fused multiply-adds
// included, so its results are theirs to the last bit: the test vectors of a hierarchy come out of
// solves with it, and a deflation's FP32 vectors magnify a last-bit change of the coarse
// operators to 1e-8 in the coarsest samples.
//
// Measured (MI355X, whole calls) against the separate launches: 8 steps with 32 deflation vectors, n =
// 1024, 32 right-hand sides 171 -> 94 us (82 in the kernel, a step 18.5 kclk: operator 11.7, of which
// 10.2 at 64 bytes per clock, dots 3.3, update 1.8); 24 steps, n = 600 with 10 dofs, 4 right-hand sides
// 421 -> 177 us (165 in the kernel: operator 6.3 kclk a step, dots 6.8, update 4.1); complex FP64, 8
// steps, n = 128 with 32 deflation vectors 187 -> 65 us.  Where a step streams more, the separate
// launches are the faster form (one_launch_mb).
#include <algorithm>

#include "coarsest.h"
#include "givens.h"
#include "wave.h"

namespace {

constexpr int CS_THREADS = 1024;
constexpr int CS_WAVES = CS_THREADS / 64;
constexpr int CS_COLS = 16;    // FP32 operator columns whose loads a thread has in flight (half in FP64)
constexpr int CS_PAD = 8;      // coefficients of zero past the last basis vector
constexpr int CS_MAX_M = 31;
// Bytes of deflation vectors that a workgroup goes through by itself: twice per right-hand side,
// at one CU's rate of 10 us a MB.  More of them take the two launches of small_deflate, about 8 us
// and as much again for 512 vectors.  Complex FP32, n = 2048, 8 steps, one right-hand side: 512
// vectors (8.4 MB) 383 us inside and 164 in launches of their own, 256 vectors 262 and 154; n =
// 1024, 256 vectors (2.1 MB) 143 and 103; about equal at 512 KB.
constexpr int64_t CS_DEFL_BYTES = 512 * 1024;
constexpr int CS_MAX_K = 128;  // vectors that these bytes can be: k <= n / 4, k n <= 65536
constexpr size_t CS_LDS = 160 * 1024;  // per workgroup

// Krylov basis of a right-hand side: vectors 0 .. kl-1 in LDS, the others in global memory
template <typename R>
struct Basis {
  Cx<R>* lds;
  Cx<R>* mem;
  int n, kl;
  __device__ __forceinline__ Cx<R>* mem_at(int i) const { return mem + (int64_t)(i - kl) * n; }
};

// f(v_i, i) for i in [i0, i1), the two parts in loops of their own (each with its address space)
#define BASIS_LOOP(B, i0, i1, UNROLL, BODY)                                     \
  {                                                                             \
    const int bl_split = min((i1), max((i0), (B).kl));                          \
    _Pragma(UNROLL) for (int i = (i0); i < bl_split; ++i) {                     \
      const auto* v = (B).lds + i * (B).n;                                      \
      BODY                                                                      \
    }                                                                           \
    _Pragma(UNROLL) for (int i = bl_split; i < (i1); ++i) {                     \
      const auto* v = (B).mem_at(i);                                            \
      BODY                                                                      \
    }                                                                           \
  }

struct SmallArgs {
  int n, d, Lx, Lt, m, k, P, nrhs;
  const void* A;
  const void* b;
  void* x;
  const void* W;        // deflation vectors [k][n] (Gamma5 X), or NULL
  const double* lam;    // (k = 0 where b is deflated already)
  int kl;               // basis vectors 0 .. kl-1 are kept in LDS
  void* basis;          // the others: [nrhs][m + 1 - kl][n]
  c128* e0;             // [nrhs][n], the deflation space's part of the solution, or NULL
};

// LDS of fixed size: constant addresses (with run-time offsets for all of them the kernel
// spilled registers).  The deflation coefficients are used before the Hessenberg matrix is.
struct SmallShared {
  union {
    c128 H[(CS_MAX_M + 1) * CS_MAX_M];
    c128 defl[2][CS_MAX_K];  // W^H b and Lambda^-1 W^H b
  };
  double stage[CS_WAVES * 64];
  c128 cf[CS_MAX_M + 1 + CS_PAD], cs[CS_MAX_M + 1 + CS_PAD], g[CS_MAX_M + 1], rs[CS_MAX_M + 1];
  double sc[CS_MAX_M + 1], rc[CS_MAX_M + 1], red[CS_WAVES];
};

// LDS sized by the level: u, w (n entries each), the split rows' partial sums, the basis
// vectors kept in LDS, the operator's blocks
template <typename R>
__host__ __device__ inline size_t small_dynamic(int n, int d, int P, int kl, bool blocks) {
  return sizeof(Cx<R>) * (size_t)n * (2 + (P > 1 ? P : 0) + kl + (blocks ? 5 * d : 0));
}

__device__ __forceinline__ void site_neighbours(int s, int Lx, int Lt, int* nb) {
  const int t = quotient(s, 1.0f / (float)Lx), x = s - t * Lx;
  nb[0] = s;
  nb[1] = (x + 1 == Lx) ? s - (Lx - 1) : s + 1;
  nb[2] = (x == 0) ? s + (Lx - 1) : s - 1;
  nb[3] = (t + 1 == Lt) ? s - (Lt - 1) * Lx : s + Lx;
  nb[4] = (t == 0) ? s + (Lt - 1) * Lx : s - Lx;
}

// the eight products of columns 2k' + h, k' = 0..3, of a lane's row in the order of the
// matrix-core stencil: step t takes dofs t, 4 + t, 8 + t, 12 + t one after the other (h = t / 2,
// v4 and m4 hold columns 4 k + 2 h and 4 k + 2 h + 1)
__device__ __forceinline__ void mfma_order(c64& acc, const float4 (&m4)[4], const float4 (&v4)[4]) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const c64 m = t ? cmk(m4[k].z, m4[k].w) : cmk(m4[k].x, m4[k].y);
      const c64 v = t ? cmk(v4[k].z, v4[k].w) : cmk(v4[k].x, v4[k].y);
      acc.x = fmaf(m.x, v.x, acc.x);
      acc.y = fmaf(m.x, v.y, acc.y);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const c64 m = t ? cmk(m4[k].z, m4[k].w) : cmk(m4[k].x, m4[k].y);
      const c64 v = t ? cmk(v4[k].z, v4[k].w) : cmk(v4[k].x, v4[k].y);
      acc.x = fmaf(-m.y, v.y, acc.x);
      acc.y = fmaf(m.y, v.x, acc.y);
    }
  }
}

// One row of the operator with PAIRS column pairs per direction, straight-line (a uniform
// branch around each load and product costs more than they do)
template <int PAIRS>
__device__ __forceinline__ c64 row_of_pairs(const float4* As, const c64* __restrict__ u, const int (&nb)[5]) {
  constexpr int d = 2 * PAIRS;
  c64 acc = cmk(0.f, 0.f);
#pragma unroll 1
  for (int dir = 0; dir < 5; ++dir) {
    const int site = dir == 0 ? nb[0] : dir == 1 ? nb[1] : dir == 2 ? nb[2] : dir == 3 ? nb[3] : nb[4];
    const float4* ud = reinterpret_cast<const float4*>(u + site * d);
    float4 m[PAIRS];
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) m[q] = As[(dir * PAIRS + q) * d];
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) {
      const float4 v = ud[q];
      cfma(acc, cmk(m[q].x, m[q].y), cmk(v.x, v.y));
      cfma(acc, cmk(m[q].z, m[q].w), cmk(v.z, v.w));
    }
  }
  return acc;
}

// The same for any number of column pairs, CS_COLS / 2 of them at a time, then those that are left
__device__ __forceinline__ c64 row_in_chunks(const float4* As, const c64* __restrict__ u, const int (&nb)[5], int d) {
  constexpr int CH = CS_COLS / 2;
  const int pairs = d / 2;
  c64 acc = cmk(0.f, 0.f);
#pragma unroll 1
  for (int dir = 0; dir < 5; ++dir) {
    const int site = dir == 0 ? nb[0] : dir == 1 ? nb[1] : dir == 2 ? nb[2] : dir == 3 ? nb[3] : nb[4];
    const float4* ud = reinterpret_cast<const float4*>(u + site * d);
    const float4* Ad = As + dir * pairs * d;
    int q0 = 0;
#pragma unroll 1
    for (; q0 + CH <= pairs; q0 += CH) {
      float4 m[CH];
#pragma unroll
      for (int q = 0; q < CH; ++q) m[q] = Ad[(q0 + q) * d];
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const float4 v = ud[q0 + q];
        cfma(acc, cmk(m[q].x, m[q].y), cmk(v.x, v.y));
        cfma(acc, cmk(m[q].z, m[q].w), cmk(v.z, v.w));
      }
    }
#pragma unroll 1
    for (; q0 < pairs; ++q0) {
      const float4 m = Ad[q0 * d], v = ud[q0];
      cfma(acc, cmk(m.x, m.y), cmk(v.x, v.y));
      cfma(acc, cmk(m.z, m.w), cmk(v.z, v.w));
    }
  }
  return acc;
}

// w = D u in complex FP32 (u, w in LDS; blocks by column pairs, in LDS or global memory), a
// thread per row, in the order of the coarse stencils; ends with a barrier
template <bool D16>
__device__ void small_op(const SmallArgs& a, const c64* A, const c64* __restrict__ u, c64* __restrict__ w, c64*) {
  const int d = D16 ? 16 : a.d, pairs = d / 2;
  for (int row = threadIdx.x; row < a.n; row += CS_THREADS) {
    const int s = D16 ? row / 16 : quotient(row, 1.0f / (float)d);
    int nb[5];
    site_neighbours(s, a.Lx, a.Lt, nb);
    // lane i of a site reads entries (i, 2 q), (i, 2 q + 1) as 16 bytes
    const float4* As = reinterpret_cast<const float4*>(A) + (int64_t)s * 5 * d * pairs + (row - s * d);
    c64 acc = cmk(0.f, 0.f);
    if constexpr (D16) {
      // (the next direction's loads ahead of this one's products spilled: slower)
#pragma unroll 1
      for (int dir = 0; dir < 5; ++dir) {
        const int site = dir == 0 ? nb[0] : dir == 1 ? nb[1] : dir == 2 ? nb[2] : dir == 3 ? nb[3] : nb[4];
        float4 m0[4], m1[4], v4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          m0[k] = As[dir * 128 + 32 * k];
          m1[k] = As[dir * 128 + 32 * k + 16];
        }
        const float4* ud = reinterpret_cast<const float4*>(u + site * 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) v4[k] = ud[2 * k];
        mfma_order(acc, m0, v4);
#pragma unroll
        for (int k = 0; k < 4; ++k) v4[k] = ud[2 * k + 1];
        mfma_order(acc, m1, v4);
      }
    } else {
      switch (pairs) {
        case 1: acc = row_of_pairs<1>(As, u, nb); break;
        case 2: acc = row_of_pairs<2>(As, u, nb); break;
        case 3: acc = row_of_pairs<3>(As, u, nb); break;
        case 4: acc = row_of_pairs<4>(As, u, nb); break;
        case 5: acc = row_of_pairs<5>(As, u, nb); break;
        case 6: acc = row_of_pairs<6>(As, u, nb); break;
        case 7: acc = row_of_pairs<7>(As, u, nb); break;
        default: acc = row_in_chunks(As, u, nb, d);
      }
    }
    w[row] = acc;
  }
  __syncthreads();
}

// The same in complex FP64 (column-major blocks), a row's columns dealt to P threads (P divides
// d): thread (site, p, i) has columns p, p + P, .. of row i, so that a site's threads read
// whole columns, and where its d P threads are lanes of one wavefront their sums meet in it
template <bool D16>
__device__ void small_op(const SmallArgs& a, const c128* A, const c128* __restrict__ u, c128* __restrict__ w,
                         c128* __restrict__ part) {
  const int d = a.d, P = a.P, site_threads = d * P, cols = d / P;
  const bool lanes = P == 1 || (site_threads <= 64 && (site_threads & (site_threads - 1)) == 0);
  for (int e = threadIdx.x; e < a.n * P; e += CS_THREADS) {  // one pass when P > 1
    const int s = quotient(e, 1.0f / (float)site_threads), rest = e - s * site_threads;
    const int p0 = quotient(rest, 1.0f / (float)d), i = rest - p0 * d;
    int nb[5];
    site_neighbours(s, a.Lx, a.Lt, nb);
    const c128* As = A + (int64_t)s * 5 * d * d + p0 * d + i;
    const c128* up = u + p0;
    c128 acc = cmk(0.0, 0.0);
    if (cols == 2) {
      c128 m[5][2];
#pragma unroll
      for (int dir = 0; dir < 5; ++dir) {
        m[dir][0] = As[dir * d * d];
        m[dir][1] = As[dir * d * d + P * d];
      }
#pragma unroll
      for (int dir = 0; dir < 5; ++dir) {
        cfma(acc, m[dir][0], up[nb[dir] * d]);
        cfma(acc, m[dir][1], up[nb[dir] * d + P]);
      }
    } else {
#pragma unroll 1
      for (int dir = 0; dir < 5; ++dir) {
        const int site = dir == 0 ? nb[0] : dir == 1 ? nb[1] : dir == 2 ? nb[2] : dir == 3 ? nb[3] : nb[4];
#pragma unroll 1
        for (int q0 = 0; q0 < cols; q0 += CS_COLS / 2) {
          c128 m[CS_COLS / 2];
#pragma unroll
          for (int t = 0; t < CS_COLS / 2; ++t)
            if (q0 + t < cols) m[t] = As[dir * d * d + (q0 + t) * P * d];
#pragma unroll
          for (int t = 0; t < CS_COLS / 2; ++t)
            if (q0 + t < cols) cfma(acc, m[t], up[site * d + (q0 + t) * P]);
        }
      }
    }
    if (lanes) {
      acc = cmk(wave::sum_lanes(acc.x, d, site_threads), wave::sum_lanes(acc.y, d, site_threads));
      if (p0 == 0) w[s * d + i] = acc;
    } else {
      part[p0 * a.n + s * d + i] = acc;
    }
  }
  if (!lanes) {
    __syncthreads();
    for (int row = threadIdx.x; row < a.n; row += CS_THREADS) {
      c128 acc = part[row];
      for (int p = 1; p < P; ++p) acc = acc + part[p * a.n + row];
      w[row] = acc;
    }
  }
  __syncthreads();
}

// <v, w> over n entries (n even, w in LDS) by a wavefront, the same value in every lane
template <typename R>
__device__ __forceinline__ c128 small_dot(const Cx<R>* v, const Cx<R>* __restrict__ w, int n) {
  struct __align__(2 * sizeof(Cx<R>)) Two {
    Cx<R> a, b;
  };
  const Two* vp = reinterpret_cast<const Two*>(v);
  const Two* wp = reinterpret_cast<const Two*>(w);
  double re = 0.0, im = 0.0;
#pragma unroll 8
  for (int p = threadIdx.x & 63; p < n / 2; p += 64) {
    const Two x = vp[p], y = wp[p];
    re = fma((double)x.a.x, (double)y.a.x, re);
    re = fma((double)x.a.y, (double)y.a.y, re);
    im = fma((double)x.a.x, (double)y.a.y, im);
    im = fma(-(double)x.a.y, (double)y.a.x, im);
    re = fma((double)x.b.x, (double)y.b.x, re);
    re = fma((double)x.b.y, (double)y.b.y, re);
    im = fma((double)x.b.x, (double)y.b.y, im);
    im = fma(-(double)x.b.y, (double)y.b.x, im);
  }
  return cmk(wave::sum(re), wave::sum(im));
}

// The exact solve on the deflation space: c = W^H b, r = b - W c and e0 = X Lambda^-1 c with
// X = Gamma5 W.  Coefficient i by a wavefront (w: b in LDS) ...
template <typename R>
__device__ __forceinline__ void defl_coefficient(const Cx<R>* W, const double* lam, const Cx<R>* __restrict__ w, int n,
                                                 int i, c128* __restrict__ c, c128* __restrict__ cl) {
  const double li = 1.0 / lam[i];
  const c128 d = small_dot(W + (int64_t)i * n, w, n);
  if ((threadIdx.x & 63) == 0) {
    c[i] = d;
    cl[i] = li * d;
  }
}

// ... and entry p of r (v: entry p of b) and of e0
template <typename R>
__device__ __forceinline__ void defl_entry(const Cx<R>* W, int n, int k, int d, int p, const c128* c, const c128* cl,
                                           c128& v, c128& e0) {
  c128 e = cmk(0.0, 0.0);
#pragma unroll 8
  for (int i = 0; i < k; ++i) {
    const Cx<R> wi = W[(int64_t)i * n + p];
    const c128 wd = cmk((double)wi.x, (double)wi.y);
    v = v - c[i] * wd;
    cfma(e, cl[i], wd);
  }
  e0 = p % d < d / 2 ? e : cmk(-e.x, -e.y);
}

// The same over many workgroups: coefficients c[r][2][k], 16 to a workgroup, then r and e0, 256
// entries to a workgroup (in the order above, so the results are the same bits)
template <typename R>
__global__ __launch_bounds__(CS_THREADS) void defl_coefficients_kernel(const Cx<R>* __restrict__ W,
                                                                       const double* __restrict__ lam,
                                                                       const Cx<R>* __restrict__ b, int n, int k,
                                                                       c128* __restrict__ c) {
  __shared__ __align__(32) Cx<R> w[SMALL_LEVEL_N];
  const int r = blockIdx.x, i = blockIdx.y * CS_WAVES + (threadIdx.x >> 6);
  for (int p = threadIdx.x; p < n; p += CS_THREADS) w[p] = b[(int64_t)r * n + p];
  __syncthreads();
  c128* cr = c + (int64_t)r * 2 * k;
  if (i < k) defl_coefficient(W, lam, w, n, i, cr, cr + k);
}

template <typename R>
__global__ __launch_bounds__(256) void defl_residual_kernel(const Cx<R>* __restrict__ W, const c128* __restrict__ c,
                                                            const Cx<R>* __restrict__ b, int n, int k, int d,
                                                            Cx<R>* __restrict__ res, c128* __restrict__ e0) {
  __shared__ c128 cs[SMALL_LEVEL_N / 2];
  const int r = blockIdx.x, p = blockIdx.y * 256 + threadIdx.x;
  for (int q = threadIdx.x; q < 2 * k; q += 256) cs[q] = c[(int64_t)r * 2 * k + q];
  __syncthreads();
  if (p >= n) return;
  const int64_t o = (int64_t)r * n + p;
  c128 v = ccast<double>(b[o]);
  defl_entry(W, n, k, d, p, cs, cs + k, v, e0[o]);
  res[o] = ccast<R>(v);
}

// red[i] = <v_i, w> for i < nb, a wavefront per basis vector, zero for the CS_PAD entries after
// them; the caller synchronises
__device__ __forceinline__ void small_dots64(const Basis<double>& V, int nb, const c128* __restrict__ w,
                                             c128* __restrict__ red) {
  for (int i = threadIdx.x >> 6; i < nb; i += CS_WAVES) {
    const c128 d = i < V.kl ? small_dot(V.lds + i * V.n, w, V.n) : small_dot(V.mem_at(i), w, V.n);
    if ((threadIdx.x & 63) == 0) red[i] = d;
  }
  if (threadIdx.x >= nb && threadIdx.x < nb + CS_PAD) red[threadIdx.x] = cmk(0.0, 0.0);
}

// Entry p of sum_i h_i v_i over i < nb; h is zero for the CS_PAD entries after them, so that the
// vectors come four (LDS; kl is a multiple of four, or past the last vector) or eight (memory)
// at a time without a branch for each, the last one once more beyond nb
__device__ __forceinline__ c128 small_combine(const Basis<double>& V, const c128* __restrict__ h, int nb, int p) {
  c128 s = cmk(0.0, 0.0);
  for (int i0 = 0; i0 < min(nb, V.kl); i0 += 4) {
#pragma unroll
    for (int i = i0; i < i0 + 4; ++i) cfma(s, h[i], V.lds[min(i, nb - 1) * V.n + p]);
  }
  for (int i0 = V.kl; i0 < nb; i0 += CS_PAD) {
#pragma unroll
    for (int i = i0; i < i0 + CS_PAD; ++i) cfma(s, h[i], V.mem_at(min(i, nb - 1))[p]);
  }
  return s;
}

// Sum of v over the workgroup, in every thread (two barriers)
__device__ __forceinline__ double small_sum(double v, double* red) {
  v = wave::sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < CS_WAVES; ++q) s += red[q];
  return s;
}

// The dots of the one-workgroup step of gram.hip on complex-FP32 vectors of at most 2048
// entries, in its order: thread t has the pair of entries 2t, 2t + 1, a wavefront tree per
// basis vector, then the wavefronts one after the other.  raw[i] = <u_i, w>; ends with a
// barrier.  stage: [CS_WAVES][64] doubles.
__device__ __forceinline__ void small_dots32(const Basis<float>& V, int nb, const c64* __restrict__ w, int n, double* stage,
                                             c128* __restrict__ raw) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int np = n / 2, nw = (np + 63) / 64;
  // wavefronts beyond the nw that cover the vectors take further groups of four basis vectors
  const int groups = CS_WAVES / nw, t = tid - (wv / nw) * nw * 64;
  if (wv < groups * nw) {
    const bool on = t < np;
    const float4 b = on ? reinterpret_cast<const float4*>(w)[t] : make_float4(0.f, 0.f, 0.f, 0.f);
    const double bx0 = b.x, by0 = b.y, bx1 = b.z, by1 = b.w;
    // eight vectors at a time where four would take a second round (all of them in LDS): n = 600,
    // 24 steps 170 -> 167 us
    if (nb > 4 * groups && V.kl >= nb) {
      for (int c0 = 8 * (wv / nw); c0 < nb; c0 += 8 * groups) {
        double acc[16];
        float4 u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = reinterpret_cast<const float4*>(V.lds + min(c0 + i, nb - 1) * n)[on ? t : 0];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          acc[2 * i] = (((double)u[i].x * bx0 + (double)u[i].y * by0) + (double)u[i].z * bx1) + (double)u[i].w * by1;
          acc[2 * i + 1] = (((double)u[i].x * by0 - (double)u[i].y * bx0) + (double)u[i].z * by1) - (double)u[i].w * bx1;
        }
        const double s = wave::sum16(acc);
        if ((lane & 3) == 0) stage[(wv % nw) * 64 + 2 * c0 + (lane >> 2)] = s;
      }
    } else {
      for (int c0 = 4 * (wv / nw); c0 < nb; c0 += 4 * groups) {
        double acc[8];
        float4 u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          u[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        // kl is a multiple of four or past the last vector: a group is in one part of the basis
        if (c0 < V.kl) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (on && c0 + i < nb) u[i] = reinterpret_cast<const float4*>(V.lds + (c0 + i) * n)[t];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (on && c0 + i < nb) u[i] = reinterpret_cast<const float4*>(V.mem_at(c0 + i))[t];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // products of two floats are exact in FP64
          acc[2 * i] = (((double)u[i].x * bx0 + (double)u[i].y * by0) + (double)u[i].z * bx1) + (double)u[i].w * by1;
          acc[2 * i + 1] = (((double)u[i].x * by0 - (double)u[i].y * bx0) + (double)u[i].z * by1) - (double)u[i].w * bx1;
        }
        const double s = wave::sum8(acc);
        if ((lane & 7) == 0) stage[(wv % nw) * 64 + 2 * c0 + (lane >> 3)] = s;
      }
    }
  }
  __syncthreads();
  if (tid < 2 * nb) {
    double s = 0.0, v[CS_WAVES];
#pragma unroll
    for (int k = 0; k < CS_WAVES; ++k) v[k] = stage[k * 64 + tid];  // (those from nw on stay unused)
#pragma unroll
    for (int k = 0; k < CS_WAVES; ++k) s = k < nw ? s + v[k] : s;
    reinterpret_cast<double*>(raw)[tid] = s;
  }
  __syncthreads();
}

// ||v||^2 of a complex-FP32 vector of at most 2048 entries in the order of the two-launch
// norm (blocks of 256 threads, one per 1024 entries), in every thread; three barriers
__device__ __forceinline__ double small_norm32(const c64* v, int n, double* red) {
  const int tid = threadIdx.x;
  const int G = (n + 1023) / 1024;
  double s = 0.0;
  if (tid < 256 * G)
    for (int p = tid; p < n; p += 256 * G) s += cabs2(v[p]);
  s = wave::sum(s);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  double t = 0.0;
  for (int g = 0; g < G; ++g) {
    double b = 0.0;
    for (int k = 0; k < 4; ++k) b += red[4 * g + k];
    t += b;
  }
  __syncthreads();
  return t;
}

template <typename R, bool LDSA, bool D16>
__global__ __launch_bounds__(CS_THREADS) void coarsest_small_kernel(SmallArgs a) {
  __shared__ __align__(32) SmallShared S;
  extern __shared__ __align__(32) unsigned char smem[];
  const int n = a.n, m = a.m, tid = threadIdx.x, r = blockIdx.x;
  Cx<R>* u = reinterpret_cast<Cx<R>*>(smem);  // the current Krylov vector
  Cx<R>* w = u + n;
  Cx<R>* part = w + n;
  Basis<R> V;
  V.lds = part + (a.P > 1 ? a.P * n : 0);
  V.mem = static_cast<Cx<R>*>(a.basis) + (int64_t)r * (m + 1 - a.kl) * n;
  V.n = n;
  V.kl = a.kl;
  Cx<R>* Al = V.lds + a.kl * n;
  auto store = [&](int i, int p, auto v) {  // entry (or pair) p of basis vector i
    using T = decltype(v);
    if (i < V.kl)
      reinterpret_cast<T*>(V.lds + i * n)[p] = v;
    else
      reinterpret_cast<T*>(V.mem_at(i))[p] = v;
    reinterpret_cast<T*>(u)[p] = v;
  };
  const Cx<R>* b = static_cast<const Cx<R>*>(a.b) + (int64_t)r * n;
  Cx<R>* x = static_cast<Cx<R>*>(a.x) + (int64_t)r * n;
  const Cx<R>* A = static_cast<const Cx<R>*>(a.A);
  if constexpr (LDSA) {
#pragma unroll 4
    for (int e = tid; e < n * 5 * a.d; e += CS_THREADS) Al[e] = A[e];
  }
  constexpr bool F32 = sizeof(R) == 4;

  // the exact solve on the deflation space (defl_coefficient, defl_entry), one pass over W for
  // the residual and e0
  const Cx<R>* W = static_cast<const Cx<R>*>(a.W);
  for (int p = tid; p < n; p += CS_THREADS) w[p] = b[p];
  __syncthreads();
  if (a.k > 0) {
    for (int i = tid >> 6; i < a.k; i += CS_WAVES) defl_coefficient(W, a.lam, w, n, i, S.defl[0], S.defl[1]);
    __syncthreads();
  }
  double nrm = 0.0;
  for (int p = tid; p < n; p += CS_THREADS) {
    c128 v = cmk((double)w[p].x, (double)w[p].y);
    if (a.k > 0) defl_entry(W, n, a.k, a.d, p, S.defl[0], S.defl[1], v, a.e0[(int64_t)r * n + p]);
    const Cx<R> u0 = ccast<R>(v);
    if (F32)
      store(0, p, u0);
    else
      u[p] = u0;
    nrm += cabs2(u0);
  }
  if constexpr (F32) {
    __syncthreads();
    nrm = small_norm32(u, n, S.red);
  } else {
    nrm = small_sum(nrm, S.red);
  }
  const double beta0 = sqrt(fmax(nrm, 0.0));
  const double inv0 = beta0 > 0.0 ? 1.0 / beta0 : 0.0;
  if (tid == 0) {
    S.g[0] = cmk(beta0, 0.0);
    S.sc[0] = F32 ? inv0 : 1.0;
  }
  if constexpr (!F32) {  // normalised basis
    for (int p = tid; p < n; p += CS_THREADS) store(0, p, inv0 * u[p]);
  }
  __syncthreads();

  for (int j = 0; j < m; ++j) {
    const int nb = j + 1;
    // the last wavefront rotates the previous column while the others stream the operator
    if (j > 0 && tid >= CS_THREADS - 64) {
      c128* prev = S.H + (j - 1) * (m + 1);
      givens_column(prev, prev[j].x, S.rc, S.rs, S.g, j - 1);
    }
    if constexpr (LDSA)
      small_op<D16>(a, Al, u, w, part);
    else
      small_op<D16>(a, A, u, w, part);
    c128* hcol = S.H + j * (m + 1);
    double bn;
    if constexpr (F32) {
      // h_i = s_j s_i <u_i, w>; u_{j+1} = s_j w - sum_i h_i s_i u_i
      small_dots32(V, nb, w, n, S.stage, S.cf);
      const double ws = S.sc[j];
      if (tid < nb) {
        const double si = S.sc[tid];
        const c128 h = cmk(ws * si * S.cf[tid].x, ws * si * S.cf[tid].y);
        hcol[tid] = h;
        S.cs[tid] = cmk(h.x * si, h.y * si);
      }
      __syncthreads();
      nrm = 0.0;
      if (2 * tid < n) {
        const float4 b0 = reinterpret_cast<const float4*>(w)[tid];
        c128 v0 = cmk(ws * (double)b0.x, ws * (double)b0.y), v1 = cmk(ws * (double)b0.z, ws * (double)b0.w);
        BASIS_LOOP(V, 0, nb, "unroll 8", {
          const float4 q = reinterpret_cast<const float4*>(v)[tid];
          const c128 h = S.cs[i];
          v0 = v0 - cprod<true>(h, cmk((double)q.x, (double)q.y));
          v1 = v1 - cprod<true>(h, cmk((double)q.z, (double)q.w));
        })
        const float4 un = make_float4((float)v0.x, (float)v0.y, (float)v1.x, (float)v1.y);
        store(nb, tid, un);
        nrm = (((double)un.x * un.x + (double)un.y * un.y) + (double)un.z * un.z) + (double)un.w * un.w;
      }
      bn = sqrt(fmax(small_sum(nrm, S.red), 0.0));
      if (tid == 0) S.sc[nb] = bn > 0.0 ? 1.0 / bn : 0.0;
    } else {
      // w' = w - V h1; h2 = V^H w'; beta^2 = ||w'||^2 - |h2|^2; v_{j+1} = (w' - V h2) / beta
      small_dots64(V, nb, w, S.cf);
      __syncthreads();
      if (tid < nb) hcol[tid] = S.cf[tid];
      nrm = 0.0;
      for (int p = tid; p < n; p += CS_THREADS) {
        const c128 wp = w[p] - small_combine(V, S.cf, nb, p);
        w[p] = wp;
        nrm += cabs2(wp);
      }
      nrm = small_sum(nrm, S.red);  // its barriers also order w' before the dots
      small_dots64(V, nb, w, S.cs);
      __syncthreads();
      const double h2n = wave::sum((tid & 63) < nb ? cabs2(S.cs[tid & 63]) : 0.0);
      if (tid < nb) hcol[tid] = hcol[tid] + S.cs[tid];
      bn = sqrt(fmax(nrm - h2n, 0.0));
      const double inv = bn > 0.0 ? 1.0 / bn : 0.0;
      for (int p = tid; p < n; p += CS_THREADS) {
        const c128 wp = w[p] - small_combine(V, S.cs, nb, p);
        store(nb, p, inv * wp);
      }
      if (tid == 0) S.sc[nb] = 1.0;
    }
    if (tid == 0) hcol[nb] = cmk(bn, 0.0);
    __syncthreads();
  }
  if (tid < 64) {
    c128* last = S.H + (m - 1) * (m + 1);
    givens_column(last, last[m].x, S.rc, S.rs, S.g, m - 1);
    __builtin_amdgcn_wave_barrier();
    // (with room for 16 columns and more in registers the kernel spilled)
    c128 y;
    if (m <= 8)
      y = givens_backsub<8>(S.H, m + 1, S.g, m);
    else
      y = givens_backsub_lds(S.H, m + 1, S.g, m);
    if (tid < m) S.g[tid] = y;
  }
  __syncthreads();
  if (tid < m) S.cf[tid] = S.sc[tid] * S.g[tid];
  __syncthreads();
  for (int p = tid; p < n; p += CS_THREADS) {
    c128 xp = cmk(0.0, 0.0);
    BASIS_LOOP(V, 0, m, "unroll 8", { xp = xp + cprod<false>(S.cf[i], cmk((double)v[p].x, (double)v[p].y)); })
    if (a.e0) xp = xp + a.e0[(int64_t)r * n + p];
    x[p] = ccast<R>(xp);
  }
}

// How a level's solve is laid out: threads that share a row's contraction, basis vectors and
// blocks in LDS
struct SmallPlan {
  int P = 1, kl = 0;
  bool blocks = false, ok = false;
  size_t shm = 0;
};

template <typename R>
SmallPlan small_plan(const Level& L, int m) {
  SmallPlan p;
  if (L.fine || m < 1 || m > CS_MAX_M || L.n() > SMALL_LEVEL_N) return p;
  const int n = (int)L.n(), d = L.dofs;
  // as many threads to a row as leave each two columns of every direction
  if (sizeof(R) == 8)
    while (2 * p.P * n <= CS_THREADS && 4 * p.P <= d && d % (2 * p.P) == 0) p.P *= 2;
  const size_t room = CS_LDS - sizeof(SmallShared);
  auto bytes = [&](int kl, bool blocks) { return small_dynamic<R>(n, d, p.P, kl, blocks); };
  if (bytes(0, false) > room) return p;
  p.ok = true;
  p.blocks = bytes(m + 1, true) <= room;
  p.kl = m + 1;
  if (bytes(p.kl, p.blocks) > room)
    for (p.kl = m / 4 * 4; bytes(p.kl, false) > room;) p.kl -= 4;
  p.shm = bytes(p.kl, p.blocks);
  return p;
}

// bytes of device scratch for the basis vectors outside LDS
template <typename R>
size_t small_scratch_bytes(const SmallPlan& p, int m, int64_t n, int nrhs) {
  return ((size_t)(m + 1 - p.kl) * nrhs * n * sizeof(Cx<R>) + 15) / 16 * 16;
}

template <typename R, bool LDSA, bool D16>
void small_launch(dmlmc_ctx* ctx, const SmallArgs& a, size_t shm) {
  auto fn = coarsest_small_kernel<R, LDSA, D16>;
  HIPCHK(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)(CS_LDS - sizeof(SmallShared))));
  hipLaunchKernelGGL(fn, dim3(a.nrhs), dim3(CS_THREADS), shm, ctx->stream, a);
  LAUNCH_CHECK();
}

}  // namespace

// Whether one launch is the faster form, from the megabytes a workgroup streams per step (blocks and
// basis vectors outside LDS, at about 10 us each) against what the separate launches take per step:
// 12 to 17 us with the matrix-core stencil (16 dofs; FP64 from 8 right-hand sides on), more with the
// scalar one, and more with many right-hand sides, of which the one launch has 256 at a time.
// Measured (us, one launch / separate, no deflation) around the lines:
//   FP32, 16 dofs, 24 steps, 1 RHS: n = 1024 (0.7 MB a step) 262 / 342, 1536 (1.1) 353 / 305, 2048 (1.6)
//     441 / 306; 32 RHS, 2048: 4 steps (1.3) 75 / 84, 24 steps 454 / 359; 128 RHS: 498 / 737
//   FP32, 24 dofs, n = 1536, 24 steps (1.6): 1 RHS 494 / 444, 2 RHS 500 / 566; 32 dofs, 2048 (2.9) 705 / 635
//   FP64, 16 dofs, 1 RHS: n = 1024, 8 steps (1.4) 148 / 152, 24 steps (1.9) 504 / 429; 2048, 24 steps (4.3)
//     934 / 380, 32 RHS 1103 / 544, 128 RHS 1428 / 1164, 512 RHS 3914 / 3788
//   FP64, 24 dofs: n = 960, 24 steps (2.4), 2 RHS 647 / 663; 1536, 8 steps (3.4), 32 RHS 293 / 246
// In complex FP32 both forms give the same bits.
double one_launch_mb(bool f32, int d, int nrhs) {
  constexpr double any = 1e9;
  if (f32) {
    if (nrhs >= 64) return any;
    if (d == 16) return nrhs < 32 ? 1.05 : 1.4;
    return nrhs > 1 ? 2.8 : d < 16 ? 0.75 : 1.55;
  }
  if (d > 16) return nrhs == 1 ? 2.1 : nrhs < 128 ? 2.8 : nrhs < 512 ? 4.1 : any;
  if (nrhs < 64) return nrhs == 1 ? 1.36 : 1.6;
  return d == 16 || nrhs < 128 ? (nrhs < 4096 ? 2.05 : any) : nrhs < 512 ? 4.1 : any;
}

template <typename R>
bool coarsest_small_ok(const Level& L, int m, int nrhs) {
  constexpr bool F32 = std::is_same<R, float>::value;
  const SmallPlan p = small_plan<R>(L, m);
  if (!p.ok) return false;
  const double vec = 1e-6 * L.n() * sizeof(Cx<R>), outside = std::max(0, m - p.kl);
  const double mb = (p.blocks ? 0.0 : vec * 5 * L.dofs * m) + vec * (F32 ? 2 : 4) * outside * (outside + 1) / 2;
  return mb <= m * one_launch_mb(F32, L.dofs, nrhs);
}

template <typename R>
bool small_deflates_inside(const Level& L, int k) {
  return k * L.n() * (int64_t)sizeof(Cx<R>) <= CS_DEFL_BYTES;
}

template <typename R>
void small_deflate(dmlmc_ctx* ctx, const Level& L, const dmlmc_defl* D, const Cx<R>* b, int nrhs, c128* c, Cx<R>* r,
                   c128* e0) {
  const int n = (int)L.n(), k = D->k;
  REQUIRE(n <= SMALL_LEVEL_N && 4 * k <= n && D->n == n, "level not laid out for the deflation of small levels");
  const Cx<R>* W = std::is_same<R, float>::value ? (const Cx<R>*)D->W32.p : (const Cx<R>*)D->W64.p;
  KTimer kt(ctx, "defl_gemm", 24.0 * n * k * nrhs);
  hipLaunchKernelGGL((defl_coefficients_kernel<R>), dim3(nrhs, (unsigned)ceil_div(k, CS_WAVES)), dim3(CS_THREADS), 0,
                     ctx->stream, W, D->lam_dev.as<double>(), b, n, k, c);
  LAUNCH_CHECK();
  hipLaunchKernelGGL((defl_residual_kernel<R>), dim3(nrhs, (unsigned)ceil_div(n, 256)), dim3(256), 0, ctx->stream, W, c,
                     b, n, k, L.dofs, r, e0);
  LAUNCH_CHECK();
}

template <typename R>
size_t coarsest_small_scratch(const Level& L, int m, int k, int nrhs) {
  return small_scratch_bytes<R>(small_plan<R>(L, m), m, L.n(), nrhs) + (k > 0 ? sizeof(c128) * nrhs * L.n() : 0);
}

template <typename R>
void coarsest_small(dmlmc_ctx* ctx, const Level& L, const dmlmc_defl* D, const Cx<R>* b, Cx<R>* x, int nrhs, int m,
                    void* scratch, c128* e0) {
  constexpr bool F32 = std::is_same<R, float>::value;
  const int k = D ? D->k : 0;
  const SmallPlan p = small_plan<R>(L, m);
  SmallArgs a;
  a.n = (int)L.n();
  a.d = L.dofs;
  a.Lx = L.Lx;
  a.Lt = L.Lt;
  a.m = m;
  a.k = k;
  a.P = p.P;
  a.nrhs = nrhs;
  a.A = F32 ? L.Apair32.p : L.A64.p;
  a.b = b;
  a.x = x;
  a.W = D ? (F32 ? D->W32.p : D->W64.p) : nullptr;
  a.lam = D ? D->lam_dev.as<double>() : nullptr;
  a.kl = p.kl;
  a.basis = scratch;
  a.e0 = D ? reinterpret_cast<c128*>(static_cast<char*>(scratch) + small_scratch_bytes<R>(p, m, L.n(), nrhs)) : e0;
  REQUIRE(p.ok && a.A != nullptr && (scratch != nullptr || (p.kl == m + 1 && k == 0)) &&
              (D == nullptr || small_deflates_inside<R>(L, k)),
          "level not laid out for the one-launch coarsest solve");
  // the operator's blocks once per step and right-hand side
  KTimer kt(ctx, "coarsest", (double)nrhs * m * 5 * L.dofs * L.n() * sizeof(Cx<R>));
  if (F32 && L.dofs == 16) {
    if (p.blocks)
      small_launch<R, true, F32>(ctx, a, p.shm);
    else
      small_launch<R, false, F32>(ctx, a, p.shm);
  } else if (p.blocks) {
    small_launch<R, true, false>(ctx, a, p.shm);
  } else {
    small_launch<R, false, false>(ctx, a, p.shm);
  }
}

#define INST(R)                                                                                                      \
  template bool coarsest_small_ok<R>(const Level&, int, int);                                                        \
  template bool small_deflates_inside<R>(const Level&, int);                                                         \
  template void small_deflate<R>(dmlmc_ctx*, const Level&, const dmlmc_defl*, const Cx<R>*, int, c128*, Cx<R>*, c128*); \
  template size_t coarsest_small_scratch<R>(const Level&, int, int, int);                                            \
  template void coarsest_small<R>(dmlmc_ctx*, const Level&, const dmlmc_defl*, const Cx<R>*, Cx<R>*, int, int, void*, \
                                  c128*);
INST(float)
INST(double)
#undef INST
