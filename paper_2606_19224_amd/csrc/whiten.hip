// Non-diagonal observation covariance R = L L^T with a lower-bidiagonal L
// (Section 5.1; the tridiagonal Toeplitz R of Section 5.3 and Example 2).
//
// The analysis whitens the observation space by L: with S~ = L^{-1} S and
// D~ = L^{-1} D the innovation system L^{-1} Psi L^{-T} (L^T z) = L^{-1} d
// has the matrix I + S~ S~^T/(N-1), and W = S^T Z/(N-1) = S~^T Z~/(N-1).  So
// the solvers run unchanged on a problem whose observations are S~ itself:
// rows X' = S~ (already centred), H = I, y' = 0, perturbations
// E' = D~ + S~ (so that y' + E' - H X' = D~) and R' = I, with the update
// applied to the real X_f.  This is CG preconditioned by M = R (the L^{-1}
// scaling of Algorithm 2 applied to the full system), exact for any R with
// such a factor.  The kernels here build that problem, map a warm start to
// the whitened variables (z~0 = L^T z0) and a solution back
// (z = L^{-T} z~), and factor a symmetric tridiagonal R.
//
// L is given as 2m-1 values: its diagonal (m), then its subdiagonal (m-1),
// e[i] = L[i+1][i].
#include "internal.h"
#include "mfma_util.h"

namespace cgd {

namespace {

constexpr int kWB = 256;

// The forward substitution x_i = (b_i - e_{i-1} x_{i-1}) / d_i =
// a_i x_{i-1} + b_i / d_i, a_i = -e_{i-1} / d_i, is a serial chain of m steps
// per member (1.66 ms at m = 4096, one thread per member, with one thread per
// row for the gather before it another 0.12 ms).  Cut into chunks of kTriRows
// rows it is a scan: every chunk is solved from x = 0 (k_tri_local, as many
// workgroups as chunks, in the launch that gathers the rows), the true last
// row of each chunk follows from the previous chunk's (k_tri_carry, m /
// kTriRows steps), and the rest of a chunk adds the previous chunk's last row
// times the running product of a (k_tri_apply).  All in double.
// 32 rows: the chunks of m = 4096 give 128 workgroups and 128 carry steps
// (n = m = 4096, N = 100, FP32: whole analysis 2062 -> 325 us).
constexpr int kTriRows = 32;
constexpr int kTriLdsN = 256;  // largest N whose chunk (2 x 32 x N doubles) is kept in LDS

// Chunk blockIdx.x: HX (double) from X_f, idx, w; S = HX - mean and D = y +
// eps - HX; then both by substitution from x = 0 into Sd and Dd.
// pend[chunk] = product of the chunk's a.  LM: HX and D sit in LDS, else in
// Sd and Dd themselves.
template <typename T, bool LM>
__global__ __launch_bounds__(kWB) void k_tri_local(int n, int m, int N, int k, const T* Xf,
                                                   const int32_t* idx, const T* hw, const T* y,
                                                   const T* eps, const T* Lf, double* Sd,
                                                   double* Dd, double* pend, int* err) {
  extern __shared__ __align__(16) double tri_sh[];
  __shared__ double dl[kTriRows], al[kTriRows], mu[kTriRows];
  const int tid = threadIdx.x, i0 = blockIdx.x * kTriRows, rows = min(kTriRows, m - i0);
  const int ne = rows * N;
  const size_t g0 = (size_t)i0 * N;
  double* hs;
  double* hd;
  if constexpr (LM) {
    hs = tri_sh;
    hd = tri_sh + (size_t)kTriRows * N;
  } else {
    hs = Sd + g0;
    hd = Dd + g0;
  }
  if (tid < kTriRows) {
    const int i = i0 + tid;
    const bool live = i < m;
    const double d = live ? (double)Lf[i] : 1.0;
    dl[tid] = d;
    al[tid] = (live && i > 0) ? -(double)Lf[m + i - 1] / d : 0.0;
  }
  constexpr int U = 4;  // elements in flight per thread
  for (int e0 = tid; e0 < ne; e0 += kWB * U) {
    double h[U], d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kWB, r = e / N;
      h[u] = 0.0;
      d[u] = e < ne && eps ? (double)eps[g0 + e] : 0.0;
    }
    for (int t = 0; t < k; ++t)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kWB, r = e / N, j = e - r * N;
        if (e < ne) {
          const size_t at = (size_t)(i0 + r) * k + t;
          const int c = idx[at];
          if ((unsigned)c < (unsigned)n)
            h[u] += (double)hw[at] * (double)Xf[(size_t)c * N + j];
          else
            atomicOr(err, 2);
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kWB, r = e / N;
      if (e < ne) {
        hs[e] = h[u];
        hd[e] = (double)y[i0 + r] - h[u] + d[u];
      }
    }
  }
  __syncthreads();
  {
    const int r = tid / 8, q = tid % 8;  // eight lanes per row
    double s = 0.0;
    if (r < rows)
      for (int j = q; j < N; j += 8) s += hs[r * N + j];
    s = group_sum<8>(s);
    if (q == 0) mu[r] = s / N;
  }
  __syncthreads();
  for (int col = tid; col < 2 * N; col += kWB) {
    const bool left = col < N;
    const int j = left ? col : col - N;
    const double* src = left ? hs : hd;
    double* out = (left ? Sd : Dd) + g0 + j;
    double x = 0.0;
    for (int r0 = 0; r0 < rows; r0 += 8) {
      double c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = r0 + u;
        c[u] = r < rows ? (src[r * N + j] - (left ? mu[r] : 0.0)) / dl[r] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = r0 + u;
        if (r < rows) {
          x = fma(al[r], x, c[u]);
          out[(size_t)r * N] = x;
        }
      }
    }
  }
  if (tid == 0) {
    double p = 1.0;
    for (int r = 0; r < rows; ++r) p *= al[r];
    pend[blockIdx.x] = p;
  }
}

// The true last row of every chunk, in order: one thread per column of S
// (then D), 16 chunks of loads in flight.
__global__ __launch_bounds__(64) void k_tri_carry(int m, int N, int nch, const double* pend,
                                                  double* Sd, double* Dd) {
  const int col = blockIdx.x * 64 + threadIdx.x;
  if (col >= 2 * N) return;
  double* a = col < N ? Sd + col : Dd + (col - N);
  constexpr int U = 16;
  double x = 0.0;
  for (int c0 = 0; c0 < nch; c0 += U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u;
      v[u] = c < nch ? a[(size_t)(min((c + 1) * kTriRows, m) - 1) * N] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u;
      if (c < nch) {
        x = c > 0 ? fma(pend[c], x, v[u]) : v[u];
        a[(size_t)(min((c + 1) * kTriRows, m) - 1) * N] = x;
      }
    }
  }
}

// Chunk blockIdx.x: X'[i][j] = S~_ij and E'[i][j] = D~_ij + S~_ij from the
// chunk's own solution, the running products of a and the previous chunk's
// last row; also the chunk's rows of the constant arrays idx' = i, w' = 1,
// y' = 0, R' = 1.
template <typename T>
__global__ __launch_bounds__(kWB) void k_tri_apply(int m, int N, const T* Lf, const double* Sd,
                                                   const double* Dd, T* Xp, T* Ep, int32_t* idxp,
                                                   T* wp, T* yp, T* rp) {
  __shared__ double pr[kTriRows];
  const int tid = threadIdx.x, i0 = blockIdx.x * kTriRows, rows = min(kTriRows, m - i0);
  if (tid < rows) {
    const int i = i0 + tid;
    pr[tid] = i > 0 ? -(double)Lf[m + i - 1] / (double)Lf[i] : 0.0;
    idxp[i] = i;
    wp[i] = (T)1;
    yp[i] = (T)0;
    rp[i] = (T)1;
  }
  __syncthreads();
  if (tid == 0) {
    for (int r = 1; r < rows; ++r) pr[r] *= pr[r - 1];
    pr[rows - 1] = 0.0;  // the last row is final
  }
  __syncthreads();
  const size_t g0 = (size_t)i0 * N;
  const double* sin = Sd + g0 - N;  // read for i0 > 0 only
  const double* din = Dd + g0 - N;
  for (int e = tid; e < rows * N; e += kWB) {
    const int r = e / N, j = e - r * N;
    double xs = Sd[g0 + e], xd = Dd[g0 + e];
    if (i0 > 0) {
      xs = fma(pr[r], sin[j], xs);
      xd = fma(pr[r], din[j], xd);
    }
    Xp[g0 + e] = (T)xs;
    Ep[g0 + e] = (T)(xd + xs);
  }
}

// Warm start in the whitened variables: z~0 = L^T z0, row i =
// d_i z0_i + e_i z0_{i+1} (the last row has no second term).
template <typename T>
__global__ __launch_bounds__(kWB) void k_tri_z0(int m, int N, const T* Lf, const T* z0, T* zt) {
  const long total = (long)m * N;
  for (long e = (long)blockIdx.x * kWB + threadIdx.x; e < total; e += (long)gridDim.x * kWB) {
    const int i = (int)(e / N);
    double v = (double)Lf[i] * (double)z0[e];
    if (i + 1 < m) v += (double)Lf[m + i] * (double)z0[e + N];
    zt[e] = (T)v;
  }
}

// A solution back from the whitened variables, in place: z = L^{-T} z~ by
// backward substitution (z_{m-1} = z~_{m-1} / d_{m-1},
// z_i = (z~_i - e_i z_{i+1}) / d_i).  One thread per member.
template <typename T>
__global__ __launch_bounds__(kWB) void k_tri_back(int m, int N, const T* Lf, T* z) {
  const int j = blockIdx.x * kWB + threadIdx.x;
  if (j >= N) return;
  double x = 0.0;
  for (int i = m - 1; i >= 0; --i) {
    const double e = i + 1 < m ? (double)Lf[m + i] : 0.0;
    x = ((double)z[(size_t)i * N + j] - e * x) / (double)Lf[i];
    z[(size_t)i * N + j] = (T)x;
  }
}

// Cholesky factor of the symmetric tridiagonal R (diagonal r, off-diagonal
// o): d_0 = sqrt(r_0), e_i = o_i / d_i, d_{i+1} = sqrt(r_{i+1} - e_i^2), in
// double.  A pivot that is not positive or not finite leaves d_0 = -1 (the
// host checks d_0); `bad` is unused.
template <typename T>
__global__ void k_tri_chol(int m, const T* r, const T* o, T* Lf, int* bad) {
  (void)bad;
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  double p = (double)r[0];
  int b = !(p > 0.0) || !isfinite(p);
  double d = sqrt(p);
  const double d0 = d;
  for (int i = 0; i + 1 < m; ++i) {
    const double e = (double)o[i] / d;
    p = (double)r[i + 1] - e * e;
    if (!(p > 0.0) || !isfinite(p)) b = 1;
    d = sqrt(p);
    Lf[m + i] = (T)e;
    Lf[i + 1] = (T)d;
  }
  Lf[0] = b ? (T)-1 : (T)d0;
}

}  // namespace

template <typename T>
hipError_t launch_tri_whiten(int n, int m, int N, int k, const T* Xf, const int32_t* idx,
                             const T* hw, const T* y, const T* eps, const T* Lf, const T* z0,
                             const TriBuffers<T>& tb, int* err, hipStream_t s) {
  hipError_t e = launch_zero_u32((unsigned*)err, 1, s);
  if (e != hipSuccess) return e;
  // the chunk products sit in zt's region until k_tri_z0 writes it (at least
  // m / kTriRows doubles for every N >= 2; regions are rounded up to 256 bytes)
  const int nch = (m + kTriRows - 1) / kTriRows;
  double* pend = tb.pend;
  if (N <= kTriLdsN) {
    const size_t lds = sizeof(double) * 2 * kTriRows * (size_t)N;
    if ((e = hipFuncSetAttribute((const void*)k_tri_local<T, true>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
        hipSuccess)
      return e;
    hipLaunchKernelGGL((k_tri_local<T, true>), dim3(nch), dim3(kWB), lds, s, n, m, N, k, Xf, idx,
                       hw, y, eps, Lf, tb.Sd, tb.Dd, pend, err);
  } else {
    hipLaunchKernelGGL((k_tri_local<T, false>), dim3(nch), dim3(kWB), 0, s, n, m, N, k, Xf, idx,
                       hw, y, eps, Lf, tb.Sd, tb.Dd, pend, err);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (nch > 1) {
    hipLaunchKernelGGL(k_tri_carry, dim3((2 * N + 63) / 64), dim3(64), 0, s, m, N, nch,
                       (const double*)pend, tb.Sd, tb.Dd);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_tri_apply<T>, dim3(nch), dim3(kWB), 0, s, m, N, Lf, (const double*)tb.Sd,
                     (const double*)tb.Dd, tb.Xp, tb.Ep, tb.idxp, tb.wp, tb.yp, tb.rp);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (z0) {
    long nb = ((long)m * N + kWB - 1) / kWB;
    if (nb > 2048) nb = 2048;
    hipLaunchKernelGGL(k_tri_z0<T>, dim3((unsigned)nb), dim3(kWB), 0, s, m, N, Lf, z0, tb.zt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

__global__ void k_or_u32(int* dst, const int* src) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && *src) atomicOr(dst, *src);
}

hipError_t launch_or_u32(int* dst, const int* src, hipStream_t s) {
  hipLaunchKernelGGL(k_or_u32, dim3(1), dim3(64), 0, s, dst, src);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tri_back(int m, int N, const T* Lf, T* z, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_back<T>, dim3((N + kWB - 1) / kWB), dim3(kWB), 0, s, m, N, Lf, z);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tri_chol(int m, const T* r, const T* o, T* Lf, int* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_chol<T>, dim3(1), dim3(64), 0, s, m, r, o, Lf, bad);
  return hipGetLastError();
}

#define CGD_TRI_INST(T)                                                                          \
  template hipError_t launch_tri_whiten<T>(int, int, int, int, const T*, const int32_t*,         \
                                           const T*, const T*, const T*, const T*, const T*,     \
                                           const TriBuffers<T>&, int*, hipStream_t);             \
  template hipError_t launch_tri_back<T>(int, int, const T*, T*, hipStream_t);                   \
  template hipError_t launch_tri_chol<T>(int, const T*, const T*, T*, int*, hipStream_t);
CGD_TRI_INST(double)
CGD_TRI_INST(float)

}  // namespace cgd
