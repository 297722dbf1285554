// Gram-Schmidt passes of the Arnoldi step, FP64 arithmetic.
//
// Two-pass form (classical Gram-Schmidt with one reorthogonalisation, FP64 basis):
//   A: h1 = V^H w                        (read V, w)
//   B: w' = w - V h1, ||w'||^2            (read V, w; write w')
//   C: h2 = V^H w', Hessenberg column, Givens rotation, residual estimate
//   D: v_{j+1} = (w' - V h2) / beta, beta^2 = ||w'||^2 - |h2|^2
// Single-pass form (complex-FP32 cycles: unnormalised FP32 basis u_i, scales s_i = 1/||u_i||):
//   A: h_i = s_i <u_i, w>                (read U, w)
//   B: u_{j+1} = w - sum_i h_i s_i u_i, ||u_{j+1}||^2, Hessenberg column, Givens, s_{j+1}
//
// Small vectors (n <= 16384, the coarsest levels) take the single-pass step in two launches
// of 16 single-wavefront workgroups per RHS and a small finish (which a fixed-count solve
// leaves to the next step's first launch), and the two-pass step in three launches.
//
// Reductions: each workgroup reduces in LDS; with one workgroup per RHS the workgroup
// finishes the pass itself, otherwise it writes partial sums and a small kernel (one
// workgroup per RHS) adds them in a fixed order.  No atomics or device-scope fences.
#include <cmath>

#include "givens.h"
#include "solver.h"
#include "wave.h"

namespace {

constexpr int NBMAX = 32;         // basis vectors per pass
constexpr int NVMAX = 2 * NBMAX;  // reduced doubles per pass

enum FinishMode { FIN_STORE = 0, FIN_SCALED = 1, FIN_CGS2 = 2, FIN_CGS1 = 3 };

struct Fin {
  int mode = FIN_STORE;
  int j = 0, m = 0, hld = 0, nrhs = 0;
  double* out = nullptr;        // FIN_STORE: nv doubles per RHS at out + r * ostride
  int ostride = 0;
  const c128* h1 = nullptr;     // FIN_CGS2: first-pass coefficients; FIN_CGS1: the coefficients
  c128* h = nullptr;            // FIN_SCALED / FIN_CGS2: where the (scaled) coefficients go
  double* scale = nullptr;      // FIN_SCALED / FIN_CGS1: [i][nrhs]
  const double* nrm2 = nullptr; // FIN_CGS2: ||w'||^2
  c128* H = nullptr;
  double* cs = nullptr;
  c128* sn = nullptr;
  c128* g = nullptr;
  double* res = nullptr;
  double* invb = nullptr;
};

// acc[0..nv) summed over the 256-thread block into red[0..nv) (LDS); all threads return
// after red is complete.
template <int NV>
__device__ void block_reduce(const double (&acc)[NV], int nv, double* lds /* [4][NVMAX] */, double* red) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    if (q < nv) {
      const double v = wave::sum(acc[q]);
      if (l == 0) lds[w * NVMAX + q] = v;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nv; q += blockDim.x)
    red[q] = lds[q] + lds[NVMAX + q] + lds[2 * NVMAX + q] + lds[3 * NVMAX + q];
  __syncthreads();
}

// Shared memory of a step's finish: the Hessenberg column and the rotations before it
struct ColumnLds {
  c128 col[NBMAX + 1], rs[NBMAX + 1], g[NBMAX + 2];
  double rc[NBMAX + 1];
};

// Completes step j of RHS r from the column in c.col[0..j] and beta (the first wavefront does
// the work, the whole block calls it): earlier rotations, a new one, g and the residual
// estimate.  Ends without a barrier.
__device__ __forceinline__ void complete_column(const Fin& f, int r, ColumnLds& c, double beta) {
  const int l = threadIdx.x, j = f.j, m = f.m;
  if (l < j) {
    c.rc[l] = f.cs[r * m + l];
    c.rs[l] = f.sn[r * m + l];
  }
  if (l == j) c.g[j] = f.g[(int64_t)r * (m + 1) + j];
  __syncthreads();
  if (l < 64) givens_column(c.col, beta, c.rc, c.rs, c.g, j);
  __syncthreads();
  if (l <= j) f.H[(int64_t)r * (m + 1) * m + (int64_t)j * (m + 1) + l] = c.col[l];
  if (l == 0) {
    f.cs[r * m + j] = c.rc[j];
    f.sn[r * m + j] = c.rs[j];
    f.g[(int64_t)r * (m + 1) + j] = c.g[j];
    f.g[(int64_t)r * (m + 1) + j + 1] = c.g[j + 1];
    f.res[r] = sqrt(fma(c.g[j + 1].x, c.g[j + 1].x, c.g[j + 1].y * c.g[j + 1].y));
  }
}

// Completes a pass for RHS r from the reduced sums red[0..nv) in LDS (whole block calls it).
__device__ void finish_pass(const Fin& f, int r, int nv, const double* red) {
  __shared__ ColumnLds c;
  const int nb = f.j + 1, l = threadIdx.x;
  switch (f.mode) {
    case FIN_STORE:
      for (int q = l; q < nv; q += blockDim.x) f.out[(int64_t)r * f.ostride + q] = red[q];
      break;
    case FIN_SCALED:
      for (int i = l; i < nb; i += blockDim.x) {
        const double sc = f.scale[(int64_t)i * f.nrhs + r];
        f.h[(int64_t)r * f.hld + i] = cmk(red[2 * i] * sc, red[2 * i + 1] * sc);
      }
      break;
    case FIN_CGS2: {
      if (l < nb) {
        const c128 b2 = cmk(red[2 * l], red[2 * l + 1]);
        f.h[(int64_t)r * f.hld + l] = b2;
        c.col[l] = f.h1[(int64_t)r * f.hld + l] + b2;
      }
      double h2n = 0.0;
      for (int i = 0; i < nb; ++i) h2n += red[2 * i] * red[2 * i] + red[2 * i + 1] * red[2 * i + 1];
      const double beta = sqrt(fmax(f.nrm2[r] - h2n, 0.0));
      complete_column(f, r, c, beta);
      if (l == 0) f.invb[r] = beta > 0.0 ? 1.0 / beta : 0.0;
      break;
    }
    case FIN_CGS1: {
      const double beta = sqrt(fmax(red[0], 0.0));
      if (l < nb) c.col[l] = f.h1[(int64_t)r * f.hld + l];
      complete_column(f, r, c, beta);
      if (l == 0) f.scale[(int64_t)nb * f.nrhs + r] = beta > 0.0 ? 1.0 / beta : 0.0;
      break;
    }
  }
}

// The reduced sums red[0..nv) of a workgroup: finish (one workgroup per RHS) or write partials.
__device__ void finish_or_partial(int nv, const double* red, double* __restrict__ part, const Fin& f, int r) {
  if (gridDim.x == 1) {
    finish_pass(f, r, nv, red);
  } else {
    double* pr = part + ((int64_t)r * gridDim.x + blockIdx.x) * nv;
    for (int q = threadIdx.x; q < nv; q += blockDim.x) pr[q] = red[q];
  }
}

template <int NV>
__device__ void reduce_or_partial(const double (&acc)[NV], int nv, double* lds, double* red, double* __restrict__ part,
                                  const Fin& f, int r) {
  block_reduce(acc, nv, lds, red);
  finish_or_partial(nv, red, part, f, r);
}

// One workgroup per RHS, value q by wavefront q mod FINISH_WAVES: lane l adds the partials of
// blocks l, l + 64, ... into four running sums (blocks l + 256 i + 64 u go to sum u, so that
// four loads are in flight and no add waits on the previous one), then the wavefront sums
// across lanes.  (One wavefront for all values took 10.6 us at 24 values, 4 blocks.)
constexpr int FINISH_WAVES = 8;

__global__ __launch_bounds__(64 * FINISH_WAVES) void partial_finish_kernel(const double* __restrict__ part, int G,
                                                                           int nv, Fin f) {
  __shared__ double red[NVMAX];
  const int r = blockIdx.x, l = threadIdx.x & 63;
  const double* base = part + (int64_t)r * G * nv;
  for (int q = threadIdx.x >> 6; q < nv; q += FINISH_WAVES) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int g = l;
    for (; g + 192 < G; g += 256) {
      s0 += base[(int64_t)g * nv + q];
      s1 += base[(int64_t)(g + 64) * nv + q];
      s2 += base[(int64_t)(g + 128) * nv + q];
      s3 += base[(int64_t)(g + 192) * nv + q];
    }
    for (; g < G; g += 64) s0 += base[(int64_t)g * nv + q];
    const double s = wave::sum((s0 + s1) + (s2 + s3));
    if (l == 0) red[q] = s;
  }
  __syncthreads();
  finish_pass(f, r, nv, red);
}

template <typename R>
struct __align__(4 * sizeof(R)) Pair {
  Cx<R> a, b;
};

// ---------------------------------------------------------------- two-pass form, n > 16384
// Workgroups of 256 threads with LONG_EL entries to a thread and pass, the basis eight vectors
// at a time (past the last one it repeats: no branch per vector).  Bound by memory on long
// vectors and by latency on a few short ones: at n = 131072, one RHS, 24 basis vectors at most,
// a dots pass took 24 us and an update 18 with 64 workgroups and a branch per vector, 5.3 and 5.1
// like this.
constexpr int LONG_EL = 2;

// lds[wavefront][q] = the wavefront's sums over its passes, then part (or the finish)
__global__ __launch_bounds__(256) void gs_dots_kernel(const c128* __restrict__ V, int nb, const c128* __restrict__ w,
                                                      int64_t n, int64_t vstride, double* __restrict__ part, Fin f) {
  __shared__ double lds[4][NVMAX];
  __shared__ double red[NVMAX];
  const int r = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const c128* wr = w + (int64_t)r * n;
  const c128* Vr = V + (int64_t)r * n;
  lds[wv][lane] = 0.0;
  for (int64_t p0 = (int64_t)blockIdx.x * (256 * LONG_EL); p0 < n; p0 += (int64_t)gridDim.x * (256 * LONG_EL)) {
    c128 b[LONG_EL];
    int64_t p[LONG_EL];
#pragma unroll
    for (int k = 0; k < LONG_EL; ++k) {
      const int64_t e = p0 + 256 * k + threadIdx.x;
      p[k] = e < n ? e : 0;
      b[k] = wr[p[k]];
      if (e >= n) b[k] = cmk(0.0, 0.0);
    }
    for (int c0 = 0; c0 < nb; c0 += 8) {
      c128 v[LONG_EL][8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const c128* vi = Vr + min(c0 + i, nb - 1) * vstride;
#pragma unroll
        for (int k = 0; k < LONG_EL; ++k) v[k][i] = vi[p[k]];
      }
      double acc[16];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[2 * i] = acc[2 * i + 1] = 0.0;
#pragma unroll
        for (int k = 0; k < LONG_EL; ++k) {
          acc[2 * i] = fma(v[k][i].y, b[k].y, fma(v[k][i].x, b[k].x, acc[2 * i]));
          acc[2 * i + 1] = fma(-v[k][i].y, b[k].x, fma(v[k][i].x, b[k].y, acc[2 * i + 1]));
        }
      }
      const double s = wave::sum16(acc);
      if ((lane & 3) == 0) lds[wv][2 * c0 + (lane >> 2)] += s;
    }
  }
  __syncthreads();
  const int nv = 2 * nb;
  if (threadIdx.x < nv) red[threadIdx.x] = (lds[0][threadIdx.x] + lds[1][threadIdx.x]) + (lds[2][threadIdx.x] + lds[3][threadIdx.x]);
  __syncthreads();
  finish_or_partial(nv, red, part, f, r);
}

// b[k] -= sum_i h_i v_i[p[k]], hs zero from nb up to a multiple of eight
__device__ __forceinline__ void long_update(c128 (&b)[LONG_EL], const int64_t (&p)[LONG_EL], const c128* __restrict__ Vr,
                                            int nb, int64_t vstride, const c128* hs) {
  for (int c0 = 0; c0 < nb; c0 += 8) {
    c128 v[LONG_EL][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const c128* vi = Vr + min(c0 + i, nb - 1) * vstride;
#pragma unroll
      for (int k = 0; k < LONG_EL; ++k) v[k][i] = vi[p[k]];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int k = 0; k < LONG_EL; ++k) b[k] = b[k] - cprod<true>(hs[c0 + i], v[k][i]);
    }
  }
}

__device__ __forceinline__ void long_coefficients(c128* hs, const c128* __restrict__ h, int nb) {
  if (threadIdx.x < NBMAX) hs[threadIdx.x] = threadIdx.x < nb ? h[threadIdx.x] : cmk(0.0, 0.0);
  __syncthreads();
}

__global__ __launch_bounds__(256) void gs_update_norm_kernel(const c128* __restrict__ V, int nb,
                                                             c128* __restrict__ w, int64_t n, int64_t vstride,
                                                             const c128* __restrict__ h, int hld,
                                                             double* __restrict__ part, Fin f) {
  __shared__ double lds[4 * NVMAX];
  __shared__ double red[NVMAX];
  __shared__ c128 hs[NBMAX];
  const int r = blockIdx.y;
  long_coefficients(hs, h + (int64_t)r * hld, nb);
  double acc[1] = {0.0};
  c128* wr = w + (int64_t)r * n;
  for (int64_t p0 = (int64_t)blockIdx.x * (256 * LONG_EL); p0 < n; p0 += (int64_t)gridDim.x * (256 * LONG_EL)) {
    c128 b[LONG_EL];
    int64_t p[LONG_EL];
#pragma unroll
    for (int k = 0; k < LONG_EL; ++k) {
      const int64_t e = p0 + 256 * k + threadIdx.x;
      p[k] = e < n ? e : 0;
      b[k] = wr[p[k]];
    }
    long_update(b, p, V + (int64_t)r * n, nb, vstride, hs);
#pragma unroll
    for (int k = 0; k < LONG_EL; ++k) {
      const int64_t e = p0 + 256 * k + threadIdx.x;
      if (e < n) {
        wr[e] = b[k];
        acc[0] += cabs2(b[k]);
      }
    }
  }
  reduce_or_partial(acc, 1, lds, red, part, f, r);
}

__global__ __launch_bounds__(256) void gs_update_store_kernel(c128* __restrict__ V, int nb,
                                                              const c128* __restrict__ w, int64_t n, int64_t vstride,
                                                              const c128* __restrict__ h, int hld,
                                                              const double* __restrict__ invb) {
  __shared__ c128 hs[NBMAX];
  const int r = blockIdx.y;
  long_coefficients(hs, h + (int64_t)r * hld, nb);
  const double sc = invb[r];
  const c128* wr = w + (int64_t)r * n;
  c128* out = V + (int64_t)nb * vstride + (int64_t)r * n;
  for (int64_t p0 = (int64_t)blockIdx.x * (256 * LONG_EL); p0 < n; p0 += (int64_t)gridDim.x * (256 * LONG_EL)) {
    c128 b[LONG_EL];
    int64_t p[LONG_EL];
#pragma unroll
    for (int k = 0; k < LONG_EL; ++k) {
      const int64_t e = p0 + 256 * k + threadIdx.x;
      p[k] = e < n ? e : 0;
      b[k] = wr[p[k]];
    }
    long_update(b, p, V + (int64_t)r * n, nb, vstride, hs);
#pragma unroll
    for (int k = 0; k < LONG_EL; ++k) {
      const int64_t e = p0 + 256 * k + threadIdx.x;
      if (e < n) out[e] = sc * b[k];
    }
  }
}

// ---------------------------------------------------------------- single-pass form kernels
// UNR element pairs per thread and pass: their loads are all issued before the first
// product, and each pair's terms are added in the order of the pairs (the sums do not
// depend on UNR; at 1024^2, four pairs per pass against one: dots 15.1 -> 14.6 ms and
// updates 20.7 -> 20.0 ms per estimate).
template <typename RW, int NBT, int UNR>
__global__ __launch_bounds__(256) void gs1_dots_kernel(const c64* __restrict__ U, int nb,
                                                       const Cx<RW>* __restrict__ w, int64_t n, int64_t vstride,
                                                       const double* __restrict__ wscale, double* __restrict__ part,
                                                       Fin f, int64_t ld) {
  __shared__ double lds[4 * NVMAX];
  __shared__ double red[NVMAX];
  const int r = blockIdx.y;
  const double ws = wscale ? wscale[r] : 1.0;
  double acc[2 * NBT];
#pragma unroll
  for (int q = 0; q < 2 * NBT; ++q) acc[q] = 0.0;
  // element pairs (n is even): 16-byte loads of the FP32 basis
  const Pair<RW>* wr = reinterpret_cast<const Pair<RW>*>(w + (int64_t)r * ld);
  const Pair<float>* Ur = reinterpret_cast<const Pair<float>*>(U + (int64_t)r * ld);
  const int64_t np = n / 2, vs = vstride / 2, S = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += UNR * S) {
    Pair<RW> bw[UNR];
    Pair<float> u[UNR][NBT];
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      const int64_t q = p + k * S < np ? p + k * S : p;
      bw[k] = wr[q];
#pragma unroll
      for (int i = 0; i < NBT; ++i)
        if (i < nb) u[k][i] = Ur[i * vs + q];
    }
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      if (p + k * S < np) {
        const double b0x = ws * bw[k].a.x, b0y = ws * bw[k].a.y, b1x = ws * bw[k].b.x, b1y = ws * bw[k].b.y;
#pragma unroll
        for (int i = 0; i < NBT; ++i) {
          if (i < nb) {
            const Pair<float> ui = u[k][i];
            acc[2 * i] += (double)ui.a.x * b0x + (double)ui.a.y * b0y + (double)ui.b.x * b1x + (double)ui.b.y * b1y;
            acc[2 * i + 1] += (double)ui.a.x * b0y - (double)ui.a.y * b0x + (double)ui.b.x * b1y - (double)ui.b.y * b1x;
          }
        }
      }
    }
  }
  reduce_or_partial(acc, 2 * nb, lds, red, part, f, r);
}

template <typename RW, int NBT, int UNR>
__global__ __launch_bounds__(256) void gs1_update_kernel(c64* __restrict__ U, int nb, const Cx<RW>* __restrict__ w,
                                                         int64_t n, int64_t vstride, const c128* __restrict__ h,
                                                         int hld, const double* __restrict__ scale, int nrhs,
                                                         const double* __restrict__ wscale, double* __restrict__ part,
                                                         Fin f, int64_t ld) {
  __shared__ double lds[4 * NVMAX];
  __shared__ double red[NVMAX];
  __shared__ c128 hs[NBMAX];
  const int r = blockIdx.y;
  const double ws = wscale ? wscale[r] : 1.0;
  if (threadIdx.x < nb) {
    const c128 hv = h[(int64_t)r * hld + threadIdx.x];
    const double sc = scale[(int64_t)threadIdx.x * nrhs + r];
    hs[threadIdx.x] = cmk(hv.x * sc, hv.y * sc);
  }
  __syncthreads();
  double acc[1] = {0.0};
  const Pair<RW>* wr = reinterpret_cast<const Pair<RW>*>(w + (int64_t)r * ld);
  const Pair<float>* Ur = reinterpret_cast<const Pair<float>*>(U + (int64_t)r * ld);
  Pair<float>* out = reinterpret_cast<Pair<float>*>(U + (int64_t)nb * vstride + (int64_t)r * ld);
  const int64_t np = n / 2, vs = vstride / 2, S = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += UNR * S) {
    Pair<RW> bw[UNR];
    Pair<float> u[UNR][NBT];
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      const int64_t q = p + k * S < np ? p + k * S : p;
      bw[k] = wr[q];
#pragma unroll
      for (int i = 0; i < NBT; ++i)
        if (i < nb) u[k][i] = Ur[i * vs + q];
    }
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      if (p + k * S < np) {
        double v0x = ws * bw[k].a.x, v0y = ws * bw[k].a.y, v1x = ws * bw[k].b.x, v1y = ws * bw[k].b.y;
#pragma unroll
        for (int i = 0; i < NBT; ++i) {
          if (i < nb) {
            const Pair<float> ui = u[k][i];
            const c128 hi = hs[i];
            v0x -= hi.x * (double)ui.a.x - hi.y * (double)ui.a.y;
            v0y -= hi.x * (double)ui.a.y + hi.y * (double)ui.a.x;
            v1x -= hi.x * (double)ui.b.x - hi.y * (double)ui.b.y;
            v1y -= hi.x * (double)ui.b.y + hi.y * (double)ui.b.x;
          }
        }
        Pair<float> st;
        st.a = cmk((float)v0x, (float)v0y);
        st.b = cmk((float)v1x, (float)v1y);
        out[p + k * S] = st;
        acc[0] += (double)st.a.x * st.a.x + (double)st.a.y * st.a.y + (double)st.b.x * st.b.x + (double)st.b.y * st.b.y;
      }
    }
  }
  reduce_or_partial(acc, 1, lds, red, part, f, r);
}

// ---------------------------------------------------------------- single-pass form, n <= 16384
// The vectors fit a workgroup of 1024 threads (element pair p belongs to thread p % 1024), and
// the sums are those of such a workgroup: each thread's pairs in order, a tree over each
// wavefront's lanes, the wavefronts one after the other.  The 16 wavefronts are workgroups of
// their own (SPLIT_WAVES x RHS of them, so that the basis streams through many CUs): one launch
// leaves the dots' partial sums, the next adds them up in the fixed order, updates the vector and
// leaves the norm's, which the step's finish (or the next step's dots launch) adds up.
// Measured over 24 steps at n = 4096, 20 RHS: the step in one workgroup per RHS took 22 us (one
// CU's L2 rate), these two launches 4.4 + 4.5 us (the update 3.7 to 5.5 with 8 to 24 vectors); at
// n = 16384, 32 RHS, 15.4 us against 5.2 + 5.4 and 4.1 for the finish.
constexpr int SPLIT_WAVES = 16;
constexpr int SPLIT_CHUNK = 8;  // basis vectors per workgroup of the dots launch

// beta = ||u_{j+1}|| from the wavefronts' sums, its scale, and column j through the Givens
// rotations (one wavefront per RHS)
__device__ __forceinline__ void split_finish(const Fin& f, int r, const double* __restrict__ npart) {
  __shared__ ColumnLds c;
  const int l = threadIdx.x, j = f.j;
  const double part = l < SPLIT_WAVES ? npart[(int64_t)r * SPLIT_WAVES + l] : 0.0;
  if (l <= j) c.col[l] = f.h[(int64_t)r * f.hld + l];
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < SPLIT_WAVES; ++k)
    sum += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(part), k),
                            __builtin_amdgcn_readlane(__double2loint(part), k));
  const double beta = sqrt(fmax(sum, 0.0));
  complete_column(f, r, c, beta);
  if (l == 0) f.scale[(int64_t)(j + 1) * f.nrhs + r] = beta > 0.0 ? 1.0 / beta : 0.0;
}

// part[(r 16 + wave) 64 + 2 i + (0: re, 1: im)] = the wavefront's sum of <u_i, w>, i in the
// chunk blockIdx.z (past the last basis vector the chunk repeats it, into places that nothing
// reads: no branch per vector).  Blocks x = 16, z = 0 (where launched) complete the previous step
// (prev) beside.  (A wavefront per 64 pairs meeting in LDS, as in the update: 5.8 us against 4.3 at
// n = 4096.)
template <typename RW>
__global__ __launch_bounds__(64) void gs1_split_dots_kernel(const c64* __restrict__ U, int nb,
                                                            const Cx<RW>* __restrict__ w, int64_t n, int64_t vstride,
                                                            double* __restrict__ part,
                                                            const double* __restrict__ npart, Fin prev, int64_t ld) {
  const int r = blockIdx.y, lane = threadIdx.x;
  if (blockIdx.x == SPLIT_WAVES) {
    if (blockIdx.z == 0) split_finish(prev, r, npart);
    return;
  }
  const int c0 = SPLIT_CHUNK * blockIdx.z;
  const Pair<RW>* wr = reinterpret_cast<const Pair<RW>*>(w + (int64_t)r * ld);
  const Pair<float>* Ur = reinterpret_cast<const Pair<float>*>(U + (int64_t)r * ld);
  const int64_t np = n / 2, vs = vstride / 2;
  const Pair<float>* Uc[SPLIT_CHUNK];
#pragma unroll
  for (int i = 0; i < SPLIT_CHUNK; ++i) Uc[i] = Ur + min(c0 + i, nb - 1) * vs;
  double acc[2 * SPLIT_CHUNK];
#pragma unroll
  for (int q = 0; q < 2 * SPLIT_CHUNK; ++q) acc[q] = 0.0;
#pragma unroll 2
  for (int64_t p = 64 * blockIdx.x + lane; p < np; p += 64 * SPLIT_WAVES) {
    const Pair<RW> b = wr[p];
    Pair<float> u[SPLIT_CHUNK];
#pragma unroll
    for (int i = 0; i < SPLIT_CHUNK; ++i) u[i] = Uc[i][p];
#pragma unroll
    for (int i = 0; i < SPLIT_CHUNK; ++i) {
      acc[2 * i] += (double)u[i].a.x * b.a.x + (double)u[i].a.y * b.a.y + (double)u[i].b.x * b.b.x +
                    (double)u[i].b.y * b.b.y;
      acc[2 * i + 1] += (double)u[i].a.x * b.a.y - (double)u[i].a.y * b.a.x + (double)u[i].b.x * b.b.y -
                        (double)u[i].b.y * b.b.x;
    }
  }
  const double s = wave::sum16(acc);
  if ((lane & 3) == 0) part[((int64_t)r * SPLIT_WAVES + blockIdx.x) * NVMAX + 2 * c0 + (lane >> 2)] = s;
}

// h_i = s_w s_i <u_i, w> from the partial sums, u_{j+1} = s_w w - sum_i h_i s_i u_i on the
// wavefront's pairs, npart[r 16 + wave] = their part of ||u_{j+1}||^2 (of the stored values).
// A wavefront per 64 pairs (q-th of the workgroup: pairs 1024 q + 64 wave ..), the basis loads
// out before the sums are ready.  NBT: the basis count rounded up to a multiple of 8; the vectors
// past the last repeat it with a coefficient of zero (no branch per vector).
template <typename RW, int NBT>
__global__ __launch_bounds__(512) void gs1_split_update_kernel(c64* __restrict__ U, int nb,
                                                               const Cx<RW>* __restrict__ w, int64_t n,
                                                               int64_t vstride, const double* __restrict__ wscale,
                                                               const double* __restrict__ part,
                                                               double* __restrict__ npart, Fin f, int64_t ld) {
  __shared__ double cf[2 * NBMAX];  // h_i s_i
  __shared__ double nq[8][64];
  const int r = blockIdx.y, lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const double ws = wscale ? wscale[r] : 1.0;
  const Pair<RW>* wr = reinterpret_cast<const Pair<RW>*>(w + (int64_t)r * ld);
  const Pair<float>* Ur = reinterpret_cast<const Pair<float>*>(U + (int64_t)r * ld);
  const int64_t np = n / 2, vs = vstride / 2, p = 64 * (SPLIT_WAVES * q + blockIdx.x) + lane;
  const int64_t pl = p < np ? p : 0;  // idle lanes load pair 0
  const Pair<RW> b = wr[pl];
  Pair<float> u[NBT];
#pragma unroll
  for (int i = 0; i < NBT; ++i) u[i] = Ur[min(i, nb - 1) * vs + pl];
  if (threadIdx.x < 2 * nb) {
    const double* pr = part + (int64_t)r * SPLIT_WAVES * NVMAX + lane;
    double v[SPLIT_WAVES];
#pragma unroll
    for (int k = 0; k < SPLIT_WAVES; ++k) v[k] = pr[k * NVMAX];
    const double sc = f.scale[(int64_t)(lane >> 1) * f.nrhs + r];
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < SPLIT_WAVES; ++k) sum += v[k];
    const double h = ws * sc * sum;
    if (blockIdx.x == 0) reinterpret_cast<double*>(f.h + (int64_t)r * f.hld)[lane] = h;
    cf[lane] = h * sc;
  } else if (threadIdx.x < 2 * NBT) {
    cf[lane] = 0.0;
  }
  __syncthreads();
  c128 v0, v1;
  {
#pragma clang fp contract(off)
    v0 = cmk(ws * b.a.x, ws * b.a.y);  // rounded, not fused into the first subtraction
    v1 = cmk(ws * b.b.x, ws * b.b.y);
  }
#pragma unroll
  for (int i = 0; i < NBT; ++i) {
    const c128 h = cmk(cf[2 * i], cf[2 * i + 1]);
    v0 = v0 - cprod<true>(h, ccast<double>(u[i].a));
    v1 = v1 - cprod<true>(h, ccast<double>(u[i].b));
  }
  Pair<float> st;
  st.a = ccast<float>(v0);
  st.b = ccast<float>(v1);
  if (p < np) reinterpret_cast<Pair<float>*>(U + (int64_t)nb * vstride + (int64_t)r * ld)[p] = st;
  const double s =
      (double)st.a.x * st.a.x + (double)st.a.y * st.a.y + (double)st.b.x * st.b.x + (double)st.b.y * st.b.y;
  nq[q][lane] = p < np ? s : 0.0;
  __syncthreads();
  if (q == 0) {  // a lane's pairs in order, then the wavefront's tree
    double nrm = 0.0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) nrm += nq[k][lane];
    nrm = wave::sum(nrm);
    if (lane == 0) npart[(int64_t)r * SPLIT_WAVES + blockIdx.x] = nrm;
  }
}

__global__ __launch_bounds__(64) void gs1_split_finish_kernel(const double* __restrict__ npart, Fin f) {
  split_finish(f, blockIdx.x, npart);
}

// ---------------------------------------------------------------- two-pass form, n <= 16384
// Passes A to D of the two-pass form in three launches of workgroups of 256 entries: the dots
// h1; then w' = w - V h1, its norm and the dots h2 = V^H w' from the basis entries still in
// registers; then v_{j+1} = (w' - V h2) / beta, one further workgroup per RHS completing the
// Hessenberg column.  Each launch adds up the one before's partial sums itself, in a fixed
// order.  Measured at n = 4096, one RHS, over 24 steps: 96 us a step as seven launches, 13 here.
constexpr int TWO_BLOCK = 256;
constexpr int TWO_PART = NVMAX + 2;  // partial sums of a workgroup: 2 nb dots (and the norm)

// lds[wavefront][2 c0 + q] = the wavefront's sum of acc[q]
__device__ __forceinline__ void two_store_sums(double (&acc)[16], int c0, double (*lds)[NVMAX + 2]) {
  const int lane = threadIdx.x & 63;
  const double s = wave::sum16(acc);
  if ((lane & 3) == 0) lds[threadIdx.x >> 6][2 * c0 + (lane >> 2)] = s;
}

// sums[q] = the G workgroups' partials of value q < nv, added in their order by four threads
// each (value q by threads q, 64 + q, ...); ends with a barrier
__device__ __forceinline__ void two_add_partials(const double* __restrict__ part, int G, int nv, double (*lds)[NVMAX + 2],
                                                 double* sums) {
  const int q = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int v = q; v < nv; v += 64) {
    double s = 0.0;
#pragma unroll 8
    for (int g = w; g < G; g += 4) s += part[(int64_t)g * TWO_PART + v];
    lds[w][v] = s;
  }
  __syncthreads();
  for (int v = threadIdx.x; v < nv; v += blockDim.x) sums[v] = (lds[0][v] + lds[1][v]) + (lds[2][v] + lds[3][v]);
  __syncthreads();
}

__global__ __launch_bounds__(TWO_BLOCK) void gs2_split_dots_kernel(const c128* __restrict__ V, int nb,
                                                                   const c128* __restrict__ w, int64_t n,
                                                                   int64_t vstride, double* __restrict__ part) {
  __shared__ double lds[4][NVMAX + 2];
  const int r = blockIdx.y, c0 = 8 * blockIdx.z;
  const int64_t p = (int64_t)blockIdx.x * TWO_BLOCK + threadIdx.x;
  const bool on = p < n;
  const int64_t o = (int64_t)r * n + (on ? p : 0);
  c128 v[8];
  const c128 b = w[o];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = V[min(c0 + i, nb - 1) * vstride + o];
  double acc[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool use = on && c0 + i < nb;
    acc[2 * i] = use ? fma(v[i].x, b.x, v[i].y * b.y) : 0.0;
    acc[2 * i + 1] = use ? fma(v[i].x, b.y, -(v[i].y * b.x)) : 0.0;
  }
  two_store_sums(acc, c0, lds);
  __syncthreads();
  const int nv = 2 * min(8, nb - c0);
  if (threadIdx.x < nv) {
    const int q = 2 * c0 + threadIdx.x;
    part[((int64_t)r * gridDim.x + blockIdx.x) * TWO_PART + q] = (lds[0][q] + lds[1][q]) + (lds[2][q] + lds[3][q]);
  }
}

// NBT: the basis count rounded up to a multiple of 8 (the vectors past the last repeat it with
// a coefficient of zero)
template <int NBT>
__global__ __launch_bounds__(TWO_BLOCK) void gs2_split_update_dots_kernel(const c128* __restrict__ V, int nb,
                                                                          c128* __restrict__ w, int64_t n,
                                                                          int64_t vstride,
                                                                          const double* __restrict__ part1,
                                                                          double* __restrict__ part2, Fin f) {
  __shared__ double lds[4][NVMAX + 2], h[NVMAX + 2];
  const int r = blockIdx.y, G = gridDim.x;
  const int64_t p = (int64_t)blockIdx.x * TWO_BLOCK + threadIdx.x;
  const bool on = p < n;
  const int64_t o = (int64_t)r * n + (on ? p : 0);
  c128 v[NBT];
  c128 b = w[o];
#pragma unroll
  for (int i = 0; i < NBT; ++i) v[i] = V[min(i, nb - 1) * vstride + o];
  if (threadIdx.x >= 2 * nb && threadIdx.x < 2 * NBT) h[threadIdx.x] = 0.0;
  two_add_partials(part1 + (int64_t)r * G * TWO_PART, G, 2 * nb, lds, h);
  if (blockIdx.x == 0 && threadIdx.x < 2 * nb) reinterpret_cast<double*>(f.h + (int64_t)r * f.hld)[threadIdx.x] = h[threadIdx.x];
#pragma unroll
  for (int i = 0; i < NBT; ++i) b = b - cprod<true>(cmk(h[2 * i], h[2 * i + 1]), v[i]);
  if (on) w[o] = b;
#pragma unroll
  for (int c0 = 0; c0 < NBT; c0 += 8) {
    if (c0 < nb) {
      double acc[16];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool use = on && c0 + i < nb;
        acc[2 * i] = use ? fma(v[c0 + i].x, b.x, v[c0 + i].y * b.y) : 0.0;
        acc[2 * i + 1] = use ? fma(v[c0 + i].x, b.y, -(v[c0 + i].y * b.x)) : 0.0;
      }
      two_store_sums(acc, c0, lds);
    }
  }
  const double nrm = wave::sum(on ? cabs2(b) : 0.0);
  __syncthreads();  // the chunks' zero sums beyond 2 nb are written
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6][2 * nb] = nrm;
  __syncthreads();
  if (threadIdx.x <= 2 * nb) {
    const int q = threadIdx.x;
    part2[((int64_t)r * G + blockIdx.x) * TWO_PART + q] = (lds[0][q] + lds[1][q]) + (lds[2][q] + lds[3][q]);
  }
}

template <int NBT>
__global__ __launch_bounds__(TWO_BLOCK) void gs2_split_store_kernel(c128* __restrict__ V, int nb,
                                                                    const c128* __restrict__ w, int64_t n,
                                                                    int64_t vstride, const double* __restrict__ part2,
                                                                    int G, Fin f) {
  __shared__ double lds[4][NVMAX + 2], h[NVMAX + 2];
  __shared__ ColumnLds col;
  const int r = blockIdx.y;
  const bool completes = blockIdx.x == (unsigned)G;
  const int64_t p = (int64_t)blockIdx.x * TWO_BLOCK + threadIdx.x;
  const bool on = !completes && p < n;
  const int64_t o = (int64_t)r * n + (on ? p : 0);
  c128 v[NBT];
  c128 b = cmk(0.0, 0.0);
  if (!completes) {
    b = w[o];
#pragma unroll
    for (int i = 0; i < NBT; ++i) v[i] = V[min(i, nb - 1) * vstride + o];
  }
  two_add_partials(part2 + (int64_t)r * G * TWO_PART, G, 2 * nb + 1, lds, h);
  const int lane = threadIdx.x & 63;
  const double h2n = wave::sum(lane < 2 * nb ? h[lane] * h[lane] : 0.0);
  const double beta = sqrt(fmax(h[2 * nb] - h2n, 0.0));
  if (completes) {
    const int l = threadIdx.x;
    if (l < nb) col.col[l] = f.h[(int64_t)r * f.hld + l] + cmk(h[2 * l], h[2 * l + 1]);
    complete_column(f, r, col, beta);
    return;
  }
  const double inv = beta > 0.0 ? 1.0 / beta : 0.0;
#pragma unroll
  for (int i = 0; i < NBT; ++i) {
    const bool use = i < nb;  // (h[2 nb] is the norm)
    b = b - cprod<true>(cmk(use ? h[2 * i] : 0.0, use ? h[2 * i + 1] : 0.0), v[i]);
  }
  if (on) V[nb * vstride + o] = inv * b;
}

// y = R^-1 g over the first k <= K columns, times scale[i][r] where given (one wavefront per RHS).
// Measured at k = 24: 15.7 us with the terms broadcast one by one, 7.3 like this.
template <int K>
__global__ __launch_bounds__(64) void solution_kernel(int k, int m, const c128* __restrict__ H,
                                                      const c128* __restrict__ g, const double* __restrict__ scale,
                                                      c128* __restrict__ y, int nrhs) {
  const int r = blockIdx.x, c = threadIdx.x;
  const double sc = scale && c < k ? scale[(int64_t)c * nrhs + r] : 1.0;
  const c128 v = givens_backsub<K>(H + (int64_t)r * (m + 1) * m, m + 1, g + (int64_t)r * (m + 1), k);
  if (c < k) y[r * m + c] = scale ? sc * v : v;
}

// Workgroups per RHS: about 8 element pairs per thread (two passes of four), at most
// 16384 / nrhs in total (bounds the partial sums; at 1024^2 against 16 pairs and 2048 in
// total: dots and updates 34.3 -> 33.1 ms per estimate).  One workgroup per RHS finishes
// the pass in the same launch.
int gs_blocks(int64_t n, int nrhs) {
  nrhs = std::max(1, nrhs);
  int64_t g = ceil_div(n, 2 * 256 * 8);
  g = std::min<int64_t>(g, std::max(1, 16384 / nrhs));
  return (int)std::max<int64_t>(1, g);
}

void launch_partial_finish(dmlmc_ctx* ctx, const double* part, int G, int nv, const Fin& f, int nrhs) {
  if (G <= 1) return;
  hipLaunchKernelGGL(partial_finish_kernel, dim3(nrhs), dim3(64 * FINISH_WAVES), 0, ctx->stream, part, G, nv, f);
  LAUNCH_CHECK();
}

Fin base_fin(const KrylovArrays& k, int j, int nrhs) {
  Fin f;
  f.j = j;
  f.m = k.m;
  f.hld = k.hld;
  f.nrhs = nrhs;
  f.H = k.H;
  f.cs = k.cs;
  f.sn = k.sn;
  f.g = k.g;
  f.res = k.res;
  f.invb = k.invb;
  return f;
}

}  // namespace

int gs_max_basis() { return NBMAX; }

// One Arnoldi step, two-pass form: orthogonalise w (FP64, [nrhs][n]) against V_0..V_j,
// update the Hessenberg column and rotations, store V_{j+1} = w / ||w||.
void arnoldi_step(dmlmc_ctx* ctx, c128* V, c128* w, int j, int64_t n, int nrhs, const KrylovArrays& k) {
  const int nb = j + 1;
  if (nb > NBMAX) throw DmlmcError(DMLMC_EINVAL, "Krylov basis larger than the Gram-Schmidt limit");
  const int64_t vstride = (int64_t)nrhs * n;
  if (n <= GS_SPLIT_MAX_N) {
    const int G = (int)ceil_div(n, TWO_BLOCK);
    const size_t parts = (size_t)nrhs * G * TWO_PART;
    ctx->scratch_dots.ensure(sizeof(double) * 2 * parts);
    double* part1 = ctx->scratch_dots.as<double>();
    double* part2 = part1 + parts;
    Fin f = base_fin(k, j, nrhs);
    f.h = k.h1;
    KTimer kt(ctx, "gs_fused", (double)nrhs * n * (3 * nb + 5) * sizeof(c128));
    hipLaunchKernelGGL(gs2_split_dots_kernel, dim3(G, nrhs, (unsigned)ceil_div(nb, 8)), dim3(TWO_BLOCK), 0,
                       ctx->stream, V, nb, w, n, vstride, part1);
    LAUNCH_CHECK();
#define GS2_SPLIT(NBT)                                                                                               \
  hipLaunchKernelGGL(gs2_split_update_dots_kernel<NBT>, dim3(G, nrhs), dim3(TWO_BLOCK), 0, ctx->stream, V, nb, w, n, \
                     vstride, part1, part2, f);                                                                      \
  LAUNCH_CHECK();                                                                                                    \
  hipLaunchKernelGGL(gs2_split_store_kernel<NBT>, dim3(G + 1, nrhs), dim3(TWO_BLOCK), 0, ctx->stream, V, nb, w, n,   \
                     vstride, part2, G, f);                                                                          \
  LAUNCH_CHECK()
    if (nb <= 8) {
      GS2_SPLIT(8);
    } else if (nb <= 16) {
      GS2_SPLIT(16);
    } else if (nb <= 24) {
      GS2_SPLIT(24);
    } else {
      GS2_SPLIT(NBMAX);
    }
#undef GS2_SPLIT
    return;
  }
  // (partial sums bounded as in gs_blocks)
  const int G = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, 256 * LONG_EL), 16384 / std::max(1, nrhs)));
  ctx->scratch_dots.ensure(sizeof(double) * (size_t)nrhs * G * NVMAX);
  double* part = ctx->scratch_dots.as<double>();
  dim3 grid(G, nrhs);
  Fin fa = base_fin(k, j, nrhs);
  fa.mode = FIN_STORE;
  fa.out = (double*)k.h1;
  fa.ostride = 2 * k.hld;
  {
    KTimer kt(ctx, "gs_dots", (double)nrhs * n * (nb * sizeof(c128) + sizeof(c128)));
    hipLaunchKernelGGL(gs_dots_kernel, grid, dim3(256), 0, ctx->stream, V, nb, w, n, vstride, part, fa);
    LAUNCH_CHECK();
    launch_partial_finish(ctx, part, G, 2 * nb, fa, nrhs);
  }
  Fin fb = base_fin(k, j, nrhs);
  fb.mode = FIN_STORE;
  fb.out = k.nrm2;
  fb.ostride = 1;
  {
    KTimer kt(ctx, "gs_update", (double)nrhs * n * (nb * sizeof(c128) + 2 * sizeof(c128)));
    hipLaunchKernelGGL(gs_update_norm_kernel, grid, dim3(256), 0, ctx->stream, V, nb, w, n, vstride, k.h1,
                       k.hld, part, fb);
    LAUNCH_CHECK();
    launch_partial_finish(ctx, part, G, 1, fb, nrhs);
  }
  Fin fc = base_fin(k, j, nrhs);
  fc.mode = FIN_CGS2;
  fc.h1 = k.h1;
  fc.h = k.h2;
  fc.nrm2 = k.nrm2;
  {
    KTimer kt(ctx, "gs_dots", (double)nrhs * n * (nb * sizeof(c128) + sizeof(c128)));
    hipLaunchKernelGGL(gs_dots_kernel, grid, dim3(256), 0, ctx->stream, V, nb, w, n, vstride, part, fc);
    LAUNCH_CHECK();
    launch_partial_finish(ctx, part, G, 2 * nb, fc, nrhs);
  }
  {
    KTimer kt(ctx, "gs_update", (double)nrhs * n * (nb * sizeof(c128) + sizeof(c128) + sizeof(c128)));
    hipLaunchKernelGGL(gs_update_store_kernel, grid, dim3(256), 0, ctx->stream, V, nb, w, n, vstride, k.h2,
                       k.hld, k.invb);
    LAUNCH_CHECK();
  }
}

// Partial sums of the split single-pass step: [nrhs][SPLIT_WAVES][NVMAX] and [nrhs][SPLIT_WAVES]
static double* split_partials(dmlmc_ctx* ctx, int nrhs) {
  ctx->scratch_dots.ensure(sizeof(double) * (size_t)nrhs * SPLIT_WAVES * (NVMAX + 1));
  return ctx->scratch_dots.as<double>();
}

void arnoldi_finish_deferred(dmlmc_ctx* ctx, double* scale, int j, int nrhs, const KrylovArrays& k) {
  Fin f = base_fin(k, j, nrhs);
  f.h = k.h1;
  f.scale = scale;
  hipLaunchKernelGGL(gs1_split_finish_kernel, dim3(nrhs), dim3(64), 0, ctx->stream,
                     split_partials(ctx, nrhs) + (size_t)nrhs * SPLIT_WAVES * NVMAX, f);
  LAUNCH_CHECK();
}

void krylov_solution(dmlmc_ctx* ctx, const KrylovArrays& k, int iters, int nrhs, const double* scale) {
  REQUIRE(iters >= 1 && iters <= NBMAX, "Krylov basis larger than the Gram-Schmidt limit");
#define SOLUTION(K) \
  hipLaunchKernelGGL(solution_kernel<K>, dim3(nrhs), dim3(64), 0, ctx->stream, iters, k.m, k.H, k.g, scale, k.y, nrhs)
  if (iters <= 8)
    SOLUTION(8);
  else if (iters <= 16)
    SOLUTION(16);
  else if (iters <= 24)
    SOLUTION(24);
  else
    SOLUTION(NBMAX);
#undef SOLUTION
  LAUNCH_CHECK();
}

double* gs_partials(dmlmc_ctx* ctx, int64_t n, int nrhs, int extra_G) {
  const int G = std::max(gs_blocks(n, nrhs), extra_G);
  ctx->scratch_dots.ensure(sizeof(double) * (size_t)nrhs * G * NVMAX);
  return ctx->scratch_dots.as<double>();
}

template <typename RW>
void arnoldi_step_cgs1(dmlmc_ctx* ctx, c64* U, double* scale, const Cx<RW>* w, int j, int64_t n, int nrhs,
                       const KrylovArrays& k, const double* wscale, int64_t ld, int dots_G, bool deferred) {
  const int nb = j + 1;
  if (nb > NBMAX) throw DmlmcError(DMLMC_EINVAL, "Krylov basis larger than the Gram-Schmidt limit");
  if (ld <= 0) ld = n;
  REQUIRE(ld >= n && ld % 2 == 0, "Gram-Schmidt vectors need an even stride of at least their length");
  const int64_t vstride = (int64_t)nrhs * ld;
  if (n <= GS_SPLIT_MAX_N) {
    Fin f = base_fin(k, j, nrhs);
    f.h = k.h1;
    f.scale = scale;
    Fin prev = f;
    prev.j = j - 1;
    const bool chained = deferred && j > 0;  // the previous step's finish rides on the dots launch
    double* part = split_partials(ctx, nrhs);
    double* npart = part + (size_t)nrhs * SPLIT_WAVES * NVMAX;
    const unsigned per_lane = (unsigned)ceil_div(n, 2 * 64 * SPLIT_WAVES);  // pairs, at most 8
    KTimer kt(ctx, "gs_fused", (double)nrhs * n * ((2 * nb + 1) * sizeof(c64) + 2 * sizeof(Cx<RW>)));
    const dim3 dgrid(SPLIT_WAVES + (chained ? 1 : 0), nrhs, (unsigned)ceil_div(nb, SPLIT_CHUNK));
    hipLaunchKernelGGL((gs1_split_dots_kernel<RW>), dgrid, dim3(64), 0, ctx->stream, U, nb, w, n, vstride, part, npart,
                       prev, ld);
    LAUNCH_CHECK();
#define GS1_SPLIT_UPDATE(NBT)                                                                                           \
  hipLaunchKernelGGL((gs1_split_update_kernel<RW, NBT>), dim3(SPLIT_WAVES, nrhs), dim3(64 * per_lane), 0, ctx->stream, \
                     U, nb, w, n, vstride, wscale, part, npart, f, ld)
    if (nb <= 8)
      GS1_SPLIT_UPDATE(8);
    else if (nb <= 16)
      GS1_SPLIT_UPDATE(16);
    else if (nb <= 24)
      GS1_SPLIT_UPDATE(24);
    else
      GS1_SPLIT_UPDATE(NBMAX);
#undef GS1_SPLIT_UPDATE
    LAUNCH_CHECK();
    if (!deferred) {
      hipLaunchKernelGGL(gs1_split_finish_kernel, dim3(nrhs), dim3(64), 0, ctx->stream, npart, f);
      LAUNCH_CHECK();
    }
    return;
  }
  REQUIRE(!deferred, "the finish of a long vector's Gram-Schmidt step is not deferred");
  const int G = gs_blocks(n, nrhs);
  double* part = gs_partials(ctx, n, nrhs, dots_G);
  dim3 grid(G, nrhs);
  Fin fa = base_fin(k, j, nrhs);
  fa.mode = FIN_SCALED;
  fa.h = k.h1;
  fa.scale = scale;
  if (dots_G > 0) {
    // the dots were formed with w (launch_wilson_dots): only their partial sums remain
    KTimer kt(ctx, "gs_dots", 0.0);
    launch_partial_finish(ctx, part, dots_G, 2 * nb, fa, nrhs);
  } else {
    KTimer kt(ctx, "gs_dots", (double)nrhs * n * (nb * sizeof(c64) + sizeof(Cx<RW>)));
    // the basis count rounded up to 4, 8, 16 or 32 sizes the registers (and occupancy)
    if (nb <= 4)
      hipLaunchKernelGGL((gs1_dots_kernel<RW, 4, 4>), grid, dim3(256), 0, ctx->stream, U, nb, w, n, vstride, wscale, part,
                         fa, ld);
    else if (nb <= 8)
      hipLaunchKernelGGL((gs1_dots_kernel<RW, 8, 2>), grid, dim3(256), 0, ctx->stream, U, nb, w, n, vstride, wscale, part,
                         fa, ld);
    else if (nb <= 16)
      hipLaunchKernelGGL((gs1_dots_kernel<RW, 16, 1>), grid, dim3(256), 0, ctx->stream, U, nb, w, n, vstride, wscale,
                         part, fa, ld);
    else
      hipLaunchKernelGGL((gs1_dots_kernel<RW, NBMAX, 1>), grid, dim3(256), 0, ctx->stream, U, nb, w, n, vstride, wscale,
                         part, fa, ld);
    LAUNCH_CHECK();
    launch_partial_finish(ctx, part, G, 2 * nb, fa, nrhs);
  }
  Fin fb = base_fin(k, j, nrhs);
  fb.mode = FIN_CGS1;
  fb.h1 = k.h1;
  fb.scale = scale;
  {
    KTimer kt(ctx, "gs_update", (double)nrhs * n * ((nb + 1) * sizeof(c64) + sizeof(Cx<RW>)));
#define GS1_UPDATE(NBT, UNR)                                                                                      \
  hipLaunchKernelGGL((gs1_update_kernel<RW, NBT, UNR>), grid, dim3(256), 0, ctx->stream, U, nb, w, n, vstride, k.h1, \
                     k.hld, scale, nrhs, wscale, part, fb, ld)
    if (nb <= 4)
      GS1_UPDATE(4, 4);
    else if (nb <= 8)
      GS1_UPDATE(8, 2);
    else if (nb <= 16)
      GS1_UPDATE(16, 1);
    else
      GS1_UPDATE(NBMAX, 1);
#undef GS1_UPDATE
    LAUNCH_CHECK();
    launch_partial_finish(ctx, part, G, 1, fb, nrhs);
  }
}

template void arnoldi_step_cgs1<float>(dmlmc_ctx*, c64*, double*, const c64*, int, int64_t, int, const KrylovArrays&,
                                       const double*, int64_t, int, bool);
template void arnoldi_step_cgs1<double>(dmlmc_ctx*, c64*, double*, const c128*, int, int64_t, int,
                                        const KrylovArrays&, const double*, int64_t, int, bool);
