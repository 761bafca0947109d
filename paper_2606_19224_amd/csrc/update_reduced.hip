// Ensemble update, CGD-EnKF-Reduced and input validation kernels (gfx950).
#include <algorithm>
#include <type_traits>

#include "modes.h"
#include "mfma_util.h"
#include "update_tile.h"

namespace cgd {

namespace {

// X_a = X_f + A W  (mode 0, Algorithm 1 with W = S^T Z/(N-1), A = X_f - xbar 1^T)
// X_a = X_f W      (mode 1, Algorithm 2)
// Each workgroup owns RBX whole rows: it stages them in LDS before writing,
// so X_a may alias X_f.  With `skip`, nothing is written when *skip has a bit of
// kErrNoW (W was never formed).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_update(int n, int N, int RBX, const T* Xf, T* Xa,
                                                   const double* Wd, int mode, const int* skip) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (skip && (*skip & kErrNoW)) return;
  double* tile = (double*)smem_raw;  // RBX * N
  double* mean = tile + (size_t)RBX * N;
  const int tid = threadIdx.x;
  const int i0 = blockIdx.x * RBX, rows = min(RBX, n - i0), ne = rows * N;
  if (rows <= 0) return;
  for (int e = tid; e < ne; e += kBlock) tile[e] = (double)Xf[(size_t)i0 * N + e];
  __syncthreads();
  if (mode == 0) {
    for (int i = tid; i < rows; i += kBlock) {
      double s = 0;
      for (int j = 0; j < N; ++j) s += tile[i * N + j];
      mean[i] = s / N;
    }
  }
  __syncthreads();
  for (int e = tid; e < ne; e += kBlock) {
    const int i = e / N, j = e - i * N;
    double acc = 0.0;
    if (mode == 0) {
      const double mu = mean[i];
      for (int kk = 0; kk < N; ++kk) acc += (tile[i * N + kk] - mu) * Wd[(size_t)kk * N + j];
      acc += tile[e];
    } else {
      for (int kk = 0; kk < N; ++kk) acc += tile[i * N + kk] * Wd[(size_t)kk * N + j];
    }
    Xa[(size_t)i0 * N + e] = (T)acc;
  }
}

// The same update for ensembles past the tiled kernels' widths (N > 128 in
// FP32, 64 in FP64): FP64 products on the 16x16x4 MFMA whatever T is.  A
// workgroup owns 16 RT whole rows, A' in LDS in double (X_f's own term is read
// again by the lane that writes it, so X_a may alias X_f), and its waves take
// 16-column tiles of W in turn; W comes from L2 straight into the MFMA's B
// operand (16 lanes read 128 consecutive bytes).  Lane group lk sums the run lk KQ .. lk KQ + KQ - 1
// of the summation index.  Bound: FP64 MFMA, 2 n N^2 flops padded to 16, busy a
// quarter of the time: too few waves cover W's latency and the tail (n = 20011,
// N = 200: 66 us, one double FMA chain per element 370 us; 13 waves a workgroup
// 74 us, W four steps ahead 85 us).
constexpr int kWideBlock = 512;

template <typename T, int RT>
__global__ __launch_bounds__(kWideBlock) void k_update_wide(int n, int N, const T* Xf, T* Xa,
                                                            const double* Wd, int mode,
                                                            const int* skip) {
  constexpr int RB = 16 * RT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (skip && (*skip & kErrNoW)) return;
  const int TJ = (N + 15) / 16, KQ = 4 * TJ, LD = 16 * TJ + 2;
  double* As = (double*)smem_raw;  // RB x LD: A', zero past n and N
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, lr = lane & 15, lk = lane >> 4;
  const int i0 = blockIdx.x * RB, rows = min(RB, n - i0);
  for (int r = wv; r < RB; r += kWideBlock / 64) {
    double sum = 0.0;
    for (int c = lane; c < 16 * TJ; c += 64) {
      const double v = (r < rows && c < N) ? (double)Xf[(size_t)(i0 + r) * N + c] : 0.0;
      As[r * LD + c] = v;
      sum += v;
    }
    if (mode == 0) {  // (the lane reads back its own elements)
      const double mu = wave_sum(sum) / N;
      for (int c = lane; c < N; c += 64) As[r * LD + c] -= mu;
    }
  }
  __syncthreads();
  for (int tj = wv; tj < TJ; tj += kWideBlock / 64) {
    const int col = tj * 16 + lr;
    const bool cv = col < N;
    const double* wcol = Wd + (size_t)(lk * KQ) * N + (cv ? col : 0);
    v4d acc[RT];
    T xo[RT][4];  // the X_f term of mode 0, requested before the products
#pragma unroll
    for (int z = 0; z < RT; ++z) {
      acc[z] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * z + frag_row<double>(lk, i);
        xo[z][i] = (mode == 0 && r < rows && cv) ? Xf[(size_t)(i0 + r) * N + col] : (T)0;
      }
    }
    double b1[4], b2[4];  // W of the next step and the one after it
    auto fetch = [&](int t0, double (&v)[4]) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        v[t] = (cv && t0 < KQ && lk * KQ + t0 + t < N) ? wcol[(size_t)(t0 + t) * N] : 0.0;
    };
    fetch(0, b1);
    fetch(4, b2);
    for (int t0 = 0; t0 < KQ; t0 += 4) {
      double bc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        bc[t] = b1[t];
        b1[t] = b2[t];
      }
      fetch(t0 + 8, b2);
      double av[RT][4];
#pragma unroll
      for (int z = 0; z < RT; ++z) load4d(As + (16 * z + lr) * LD + lk * KQ + t0, av[z]);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int z = 0; z < RT; ++z) acc[z] = mfma4(av[z][t], bc[t], acc[z]);
    }
#pragma unroll
    for (int z = 0; z < RT; ++z)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * z + frag_row<double>(lk, i);
        if (r < rows && cv)
          Xa[(size_t)(i0 + r) * N + col] = (T)((double)xo[z][i] + acc[z][i]);
      }
  }
}

// LDS of a k_update_wide workgroup, and the launch (false: it does not fit).
template <typename T>
size_t update_wide_lds(int N, int RT) {
  return sizeof(double) * (size_t)(16 * RT) * (((N + 15) / 16) * 16 + 2);
}
constexpr size_t kUpdWideLds = 128 * 1024;

template <typename T, int RT>
hipError_t launch_update_wide(int n, int N, const T* Xf, T* Xa, const double* Wd, int mode,
                              const int* skip, hipStream_t s) {
  const size_t lds = update_wide_lds<T>(N, RT);
  const hipError_t e = hipFuncSetAttribute((const void*)k_update_wide<T, RT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_update_wide<T, RT>), dim3((n + 16 * RT - 1) / (16 * RT)),
                     dim3(kWideBlock), lds, s, n, N, Xf, Xa, Wd, mode, skip);
  return hipGetLastError();
}

// The same update on the 16x16x4 MFMA for N <= 128 (FP32) or N <= 64 (FP64),
// 64-row tiles (see update_tile.h): each workgroup brings W into LDS once
// and then takes every gridDim.x-th tile.
template <typename T, int NP>
__global__ __launch_bounds__(kBlock) void k_update_mfma(int n, int N, const T* Xf, T* Xa,
                                                        const double* Wd, int mode,
                                                        const int* skip) {
  using C = UCfg<T, NP>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (skip && (*skip & kErrNoW)) return;
  T* Wt = (T*)smem_raw;
  T* As = Wt + (size_t)NP * C::LD;
  T* Xr = As + (size_t)C::RBX * C::LD;
  double* mean = (double*)(Xr + (size_t)C::RBX * C::LD);
  update_load_w<T, NP, kBlock>(N, Wd, mode, Wt);
  update_tiles_stream<T, NP, kBlock, C::RBX>(n, N, Xf, Xa, mode, As, mode == 0 ? Xr : As, Wt, mean);
}

// The same update with the A' operand read from global memory straight into
// the MFMA's registers: no tile of X_f passes through LDS and no barrier is
// taken per tile.  W'^T sits in LDS (from Wd as update_load_w forms it, or, WT,
// already transposed in T as k_red_update takes it, of row stride WS).  Each
// wave takes 16-row blocks in turn over the whole grid (workgroups first, then
// their waves); lane (lr, lk) holds row lr's columns 4 VU s + VU lk + u, the
// permutation of the summation index the B operand uses too, so that a load
// instruction reads 64 consecutive bytes of each row (16-byte loads: N a
// multiple of VU = 16/sizeof(T), X_f and X_a 16-byte aligned).  (Runs of NP/4
// columns per lane fetched each 128-byte line eight times, past the L1: 98 us
// against 71 us at n = 10^5, N = 100 in FP64, padded to 112 as well; 36 against 33 us
// at n = 65536, N = 128 in FP32.)  NP is N rounded up to 16 here.  Mode 0
// centres each row with its mean (the lane's part plus two shuffles across the
// row's four lanes).  X_f is read again for the output elements before the
// block's stores, so X_a may alias X_f.
constexpr int kUpdWaves = 8;

template <typename T, int NP, bool WT>
__global__ __launch_bounds__(64 * kUpdWaves) void k_update_rows(int n, int N, int WS, const T* Xf,
                                                               T* Xa, const double* Wd,
                                                               const T* Wtg, int mode,
                                                               const int* skip) {
  using U = UCfg<T, NP>;
  constexpr int VU = 16 / (int)sizeof(T), BS = 64 * kUpdWaves;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (skip && (*skip & kErrNoW)) return;
  T* Wt = (T*)smem_raw;  // NP x LD
  const int tid = threadIdx.x, wv = tid >> 6;
  if constexpr (WT) {
    constexpr int NC = NP * NP / VU, UL = 8;  // 16-byte chunks, loads in flight per thread
    for (int e0 = tid; e0 < NC; e0 += BS * UL) {
      T v[UL][VU];
#pragma unroll
      for (int u = 0; u < UL; ++u) {
        const int e = e0 + u * BS, row = e / (NP / VU), c = (e - row * (NP / VU)) * VU;
        if (e < NC) vload<VU>(Wtg + (size_t)row * WS + c, v[u]);
      }
#pragma unroll
      for (int u = 0; u < UL; ++u) {
        const int e = e0 + u * BS, row = e / (NP / VU), c = (e - row * (NP / VU)) * VU;
        if (e < NC)
#pragma unroll
          for (int q = 0; q < VU; ++q) Wt[row * U::LD + c + q] = v[u][q];
      }
    }
  } else {
    update_load_w<T, NP, BS>(N, Wd, mode, Wt);
  }
  __syncthreads();
  // blocks go round the workgroups first, then their waves, so that a small n
  // still spreads over the whole grid
  const int nb = (n + 15) / 16, step = gridDim.x * kUpdWaves;
  for (int b = blockIdx.x + gridDim.x * wv; b < nb; b += step) {
    T av[NP / 4];
    update_block_load<T, NP>(n, N, Xf, b, av);
    update_block_rows<T, NP>(n, N, Xf, Xa, mode, b, av, Wt);
  }
}

// Whether k_update_rows applies and pays: N a multiple of the 16-byte vector,
// both arrays 16-byte aligned, and enough 16-row blocks that a full grid of
// 8-wave workgroups gives every wave one (n >= 32768 on 256 CUs).  Below that
// the LDS-tiled updates, which share a tile among four waves, measured
// faster (twin workload, n = 4096: 25985 against about 28000 reduced analyses/s).
constexpr int kUpdRowsMinN = 16 * kUpdWaves * 256;
template <typename T>
bool update_rows_ok(int n, int N, const T* Xf, const T* Xa) {
  return n >= kUpdRowsMinN && N % (16 / (int)sizeof(T)) == 0 && ((uintptr_t)Xf & 15) == 0 &&
         ((uintptr_t)Xa & 15) == 0;
}

template <typename T, int NP, bool WT>
hipError_t launch_update_rows_np(int n, int N, int WS, const T* Xf, T* Xa, const double* Wd,
                                 const T* Wt, int mode, const int* skip, hipStream_t s) {
  using U = UCfg<T, NP>;
  constexpr size_t lds = sizeof(T) * (size_t)NP * U::LD;
  const void* fn = (const void*)k_update_rows<T, NP, WT>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // as many workgroups as run at once (each loads W' once), at most one per block
  static int resident = 0;
  if (resident == 0) {
    int dev = 0, cus = 0, per = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
        hipSuccess)
      return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_update_rows<T, NP, WT>,
                                                          64 * kUpdWaves, lds)) != hipSuccess)
      return e;
    resident = per * cus > 0 ? per * cus : 1;
  }
  const int nb = (n + 15) / 16;
  const int grid = nb < resident ? nb : resident;
  hipLaunchKernelGGL((k_update_rows<T, NP, WT>), dim3(grid), dim3(64 * kUpdWaves), lds, s, n, N,
                     WS, Xf, Xa, Wd, Wt, mode, skip);
  return hipGetLastError();
}

// N <= 128 padded to 16, 32, 48, 64, 96, 112 or 128 (the products' cost goes
// with the square of it); WS: row stride of Wt (WT only).
template <typename T, bool WT>
hipError_t launch_update_rows(int n, int N, int WS, const T* Xf, T* Xa, const double* Wd,
                              const T* Wt, int mode, const int* skip, hipStream_t s) {
#define CGD_UPD_NP(NP) \
  if (N <= NP) return launch_update_rows_np<T, NP, WT>(n, N, WS, Xf, Xa, Wd, Wt, mode, skip, s)
  CGD_UPD_NP(16);
  CGD_UPD_NP(32);
  CGD_UPD_NP(48);
  CGD_UPD_NP(64);
  CGD_UPD_NP(96);
  CGD_UPD_NP(112);
#undef CGD_UPD_NP
  return launch_update_rows_np<T, 128, WT>(n, N, WS, Xf, Xa, Wd, Wt, mode, skip, s);
}

template <typename T, int NP>
hipError_t launch_update_mfma(int n, int N, const T* Xf, T* Xa, const double* Wd, int mode,
                              const int* skip, hipStream_t s) {
  using C = UCfg<T, NP>;
  const void* fn = (const void*)k_update_mfma<T, NP>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::lds_xr);
  if (e != hipSuccess) return e;
  // as many workgroups as run at once (each loads W once), at most one per tile
  static int resident = 0;
  if (resident == 0) {
    int dev = 0, cus = 0, per = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
        hipSuccess)
      return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_update_mfma<T, NP>, kBlock,
                                                          C::lds_xr)) != hipSuccess)
      return e;
    resident = per * cus > 0 ? per * cus : 1;
  }
  const int tiles = (n + C::RBX - 1) / C::RBX;
  const int grid = tiles < resident ? tiles : resident;
  hipLaunchKernelGGL((k_update_mfma<T, NP>), dim3(grid), dim3(kBlock), C::lds_xr, s, n, N, Xf,
                     Xa, Wd, mode, skip);
  return hipGetLastError();
}

__device__ inline double bsum(double v, double* red) {
  const int tid = threadIdx.x;
  __syncthreads();
  red[tid] = v;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  const double o = red[0];
  __syncthreads();
  return o;
}

// Final status of one column of the N x N CG: a non-finite coefficient or
// residual, else converged when the residual test holds (also on the last
// allowed step, and for b_j = 0), else stopped at maxit.
__device__ inline int small_cg_status(bool nonfinite, double rho, double thr) {
  if (nonfinite || !isfinite(rho)) return COL_NONFINITE;
  if (rho == 0.0 || sqrt(rho) <= thr) return COL_CONVERGED;
  return COL_MAXIT;
}

// CGD-EnKF-Reduced solve: one workgroup per column j of B runs textbook CG
// on the N x N SPD system G w = b_j from w = 0 (Lemma 1: at most N steps in
// exact arithmetic).  Vectors live in LDS; G is read from L2 (symmetric, so
// q_k = sum_l G[l][k] p_l reads rows coalesced).
__global__ __launch_bounds__(kBlock) void k_small_cg(int N, const double* G, const double* B,
                                                     double* W, int* iters, int* iters2,
                                                     int* status, double tol, int maxit) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* x = (double*)smem_raw;
  double* r = x + N;
  double* p = r + N;
  double* q = p + N;
  double* red = q + N;
  const int tid = threadIdx.x, j = blockIdx.x;
  double part = 0;
  for (int kk = tid; kk < N; kk += kBlock) {
    const double b = B[(size_t)kk * N + j];
    x[kk] = 0;
    r[kk] = b;
    p[kk] = b;
    part += b * b;
  }
  double rho = bsum(part, red);
  const double thr = tol * sqrt(rho);
  int it = 0;
  bool nonfinite = false;
  while (sqrt(rho) > thr && it < maxit && rho > 0.0) {
    part = 0;
    for (int kk = tid; kk < N; kk += kBlock) {
      double acc = 0;
      for (int l = 0; l < N; ++l) acc += G[(size_t)l * N + kk] * p[l];
      q[kk] = acc;
      part += p[kk] * acc;
    }
    const double pq = bsum(part, red);
    const double alpha = rho / pq;
    part = 0;
    for (int kk = tid; kk < N; kk += kBlock) {
      x[kk] += alpha * p[kk];
      r[kk] -= alpha * q[kk];
      part += r[kk] * r[kk];
    }
    const double rho_new = bsum(part, red);
    const double beta = rho_new / rho;
    for (int kk = tid; kk < N; kk += kBlock) p[kk] = r[kk] + beta * p[kk];
    __syncthreads();
    rho = rho_new;
    ++it;
    if (!isfinite(alpha) || !isfinite(beta)) {
      nonfinite = true;
      break;
    }
  }
  for (int kk = tid; kk < N; kk += kBlock) W[(size_t)kk * N + j] = x[kk];
  if (tid == 0) {
    iters[j] = it;
    if (iters2) iters2[j] = it;
    status[j] = small_cg_status(nonfinite, rho, thr);
  }
}

// ---------------------------------------------------------------------------
// Reduced mode on the MFMA, N <= 128 (Algorithm 2 with the formation costs of
// Table 2).  NP is N rounded up to 32, 64 or 128; Q is mpad x 2 NP (mpad = m
// rounded up to 32), row i = [P_i | Yt_i] with
//   P_i  = (HX_i - zbar_i 1^T) / l_i,  Yt_i = (y_i - zbar_i + E_i) / l_i,
//   l_i  = sqrt((N-1) r_i),  zbar_i = HX_i 1 / N,
// zero in the padding columns and rows.  [P^T P | P^T Yt] = Q[:, :NP]^T Q is
// a tall-skinny product over the m rows, summed in parts over row chunks
// that a later launch adds in a fixed order, with the identity.  Q is built in
// LDS, 32 rows at a time, and multiplied there: by one workgroup per 32 rows
// (k_red_pg) while N <= 64 and those are few (red_streamed), else by 256 persistent
// workgroups that add their chunks up (k_red_stream).
// ---------------------------------------------------------------------------

template <int NP> struct RedCfg {
  static constexpr int QW = 2 * NP;
  static constexpr int LPR = NP / 4;              // prep: lanes per row, 4 columns each
  static constexpr int RPB = kBlock / LPR;        // prep: rows per workgroup
};

// Gather and product in one launch for NP <= 64.  Workgroup s builds rows
// s KC .. s KC + KC - 1 of Q in LDS (zero past m), stored by column (a run of
// KC rows per column, padded to spread the banks), then forms its part of
// Q[:, :NP]^T Q on the MFMA: each wave a quarter of the NP x 2NP output, the
// summation over the chunk's rows split into four runs of KC/4, one per lane
// group (the same bijection for both operands).  Every workgroup writes its
// error word errw[s] (2: an index out of range, else 0), so no word needs
// clearing beforehand.
// SEN: the sEnKF's row scaling, l_i^2 = ||s_i||^2 + (N-1) r_i (the i-th diagonal
// entry of Zhat Zhat^T + (N-1) R), Yt = (Y - HX) / l, and only the right half
// Q[:, :NP]^T Q[:, NP:] (each wave a quarter of it).
constexpr int kRedFusedRows = 32;  // KC of the fused launch

template <typename T, int NP, bool SEN>
__global__ __launch_bounds__(kBlock) void k_red_pg(int n, int m, int N, int k, const T* Xf,
                                                   const int32_t* idx, const T* hw, const T* y,
                                                   const T* rdiag, const T* eps, T* part,
                                                   int* errw) {
  using C = RedCfg<NP>;
  using V = typename Vec4<T>::type;
  constexpr int KC = kRedFusedRows, KQ = KC / 4, LQ = KC + 16 / (int)sizeof(T);
  constexpr int PASS = KC / C::RPB;                 // rows per thread
  constexpr int MA = NP / 32, MB = SEN ? NP / 32 : NP / 16;  // 16x16 blocks per wave (a, b)
  static_assert(PASS * C::RPB == KC && KQ % 4 == 0, "chunk shape");
  __shared__ __align__(16) T qt[2 * NP * LQ];
  __shared__ int bad;
  const int tid = threadIdx.x, q = tid % C::LPR, rw = tid / C::LPR;
  const int r0 = blockIdx.x * KC;
  if (tid == 0) bad = 0;
  __syncthreads();
  // ---- Q rows of the chunk: every load of the thread's rows first ----
  double yv[PASS], rv[PASS], ev[PASS][4], h[PASS][4];
#pragma unroll
  for (int u = 0; u < PASS; ++u) {
    const int i = r0 + u * C::RPB + rw;
    const bool live = i < m;
    yv[u] = live ? (double)y[i] : 0.0;
    rv[u] = live ? (double)rdiag[i] : 1.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      h[u][c] = 0.0;
      ev[u][c] = (live && eps && 4 * q + c < N) ? (double)eps[(size_t)i * N + 4 * q + c] : 0.0;
    }
  }
  for (int t = 0; t < k; ++t) {
    int col[PASS];
    double wt[PASS];
#pragma unroll
    for (int u = 0; u < PASS; ++u) {
      const int i = r0 + u * C::RPB + rw;
      col[u] = 0;
      wt[u] = 0.0;
      if (i < m) {
        const int cx = idx[(size_t)i * k + t];
        if ((unsigned)cx < (unsigned)n) {
          col[u] = cx;
          wt[u] = (double)hw[(size_t)i * k + t];
        } else if (q == 0) {
          atomicOr(&bad, 2);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < PASS; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (4 * q + c < N) h[u][c] += wt[u] * (double)Xf[(size_t)col[u] * N + 4 * q + c];
  }
#pragma unroll
  for (int u = 0; u < PASS; ++u) {
    const int i = r0 + u * C::RPB + rw, rr = u * C::RPB + rw;
    const bool live = i < m;
    const double zb = group_sum<C::LPR>((h[u][0] + h[u][1]) + (h[u][2] + h[u][3])) / N;
    double l2 = (double)(N - 1) * rv[u];
    if constexpr (SEN) {
      double ss = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (4 * q + c < N) ss += (h[u][c] - zb) * (h[u][c] - zb);
      l2 += group_sum<C::LPR>(ss);
    }
    const double l = sqrt(l2), yz = yv[u] - zb;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = 4 * q + c;
      double pm = 0.0, yt = 0.0;
      if (live && j < N) {
        pm = (h[u][c] - zb) / l;
        yt = (yz + ev[u][c] - (SEN ? h[u][c] - zb : 0.0)) / l;
      }
      qt[j * LQ + rr] = (T)pm;
      qt[(NP + j) * LQ + rr] = (T)yt;
    }
  }
  __syncthreads();
  if (tid == 0) errw[blockIdx.x] = bad;
  // ---- the chunk's part of the product ----
  const int lane = tid & 63, wv = tid >> 6, lr = lane & 15, lk = lane >> 4;
  const int a0 = (wv >> 1) * (NP / 2), b0 = SEN ? NP + (wv & 1) * (NP / 2) : (wv & 1) * NP;
  T av[MA][KQ], bv[MB][KQ];
#pragma unroll
  for (int x = 0; x < MA; ++x) vload<KQ>(qt + (a0 + 16 * x + lr) * LQ + lk * KQ, av[x]);
#pragma unroll
  for (int z = 0; z < MB; ++z) vload<KQ>(qt + (b0 + 16 * z + lr) * LQ + lk * KQ, bv[z]);
  V acc[MA][MB];
#pragma unroll
  for (int x = 0; x < MA; ++x)
#pragma unroll
    for (int z = 0; z < MB; ++z) acc[x][z] = V{0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < KQ; ++u)
#pragma unroll
    for (int x = 0; x < MA; ++x)
#pragma unroll
      for (int z = 0; z < MB; ++z) acc[x][z] = mfma4(av[x][u], bv[z][u], acc[x][z]);
  T* out = part + (size_t)blockIdx.x * NP * C::QW;
#pragma unroll
  for (int x = 0; x < MA; ++x)
#pragma unroll
    for (int z = 0; z < MB; ++z)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out[(size_t)(a0 + 16 * x + frag_row<T>(lk, i)) * C::QW + b0 + 16 * z + lr] = acc[x][z][i];
}

// Gather and product in one persistent launch (TN = N / 16 rounded up), so that
// neither Q nor a part per 32 rows goes to memory.  Workgroup s takes the chunks s,
// s + gridDim.x, .. of 32 observation rows: it builds a chunk of Q in one of
// two LDS buffers, stored by column as in k_red_pg, and multiplies it there;
// each wave keeps its share of the output's 16 x 16 tiles (the upper tiles of
// the symmetric left half, every tile of the right half) until the last chunk.  FP32
// chains don't grow with m: up to N = 64 a chunk's product is added to its tile's sum
// in double, past that (where those sums would spill) a workgroup takes at most
// kRsChain chunks.  A chunk's indices are requested two chunks ahead and its rows one
// chunk ahead, under the previous chunk's
// products.  Thread q of a row takes the members q, q + 32, .. (coalesced reads; its
// LDS stores fall on distinct banks).  part[s][tile][16][16] in RsPart; errw and
// SEN (right half only) as in k_red_pg.
// Bound: the MFMA in FP64, the gather's latency in FP32.  At m = 10^5, N =
// 100 in FP64 the two launches this replaces, with 205 MB of Q between them,
// took 119 + 171 us, this one 119 us; at m = 16384, N = 128, k = 4 in FP32 (the
// right half) 20 + 18 us and 23 us.  (Waves that gather while others multiply,
// or the two waves of a SIMD in opposite order, ran out of registers.)
constexpr int kRsRows = 32, kRsThreads = 512, kRsWaves = kRsThreads / 64;
constexpr int kRsGroups = 256;  // one workgroup per CU

// Past N = 64 always; below, once there are more chunks than workgroups, where
// a part per chunk costs more than it spreads: at once in FP64 and for the sEnKF (N =
// 64, m = 8300: 41.2 against 39.5 us and 25.4 against 20.9), in FP32, whose streamed
// parts are in double, half as many chunks later (31.1 and 33.6 us at m = 8300, 35.9 and
// 36.2 at 12000, 45.9 and 42.0 at 20000; N = 32: 24.1 / 24.8, 26.2 / 25.9).
inline bool red_streamed(int m, int N, int esz, bool sen) {
  const int most = esz == 4 && !sen ? kRsGroups * 3 / 2 : kRsGroups;
  return N > 64 || (m + kRsRows - 1) / kRsRows > most;
}
// TN at N (as launch_red_stream chooses): two at least.
inline int red_stream_tiles(int N) { return N <= 32 ? 2 : (N + 15) / 16; }

// TS workgroups share a chunk's tiles, each building the chunk for itself: with few
// chunks one workgroup's tiles are the time (N = 128, whole reduced call, one and four
// workgroups a chunk: m = 8 28.7 and 26.1 us, m = 600 45.5 and 42.0; FP64 35.7 and 30.5,
// 61.4 and 56.5).  Past 64 chunks there are workgroups enough.
template <int TN, bool SEN, int TS>
struct RsCfg {
  static constexpr int NTL = SEN ? 0 : TN * (TN + 1) / 2;  // left tiles
  static constexpr int NT = NTL + TN * TN;
  static constexpr int TPW = (NT + TS * kRsWaves - 1) / (TS * kRsWaves);  // tiles per wave
};
constexpr int kRsSplit = 4;
inline bool red_stream_split(int m, int N) {
  return N > 64 && (m + kRsRows - 1) / kRsRows * kRsSplit <= kRsGroups;
}
// FP32, N <= 64: sums and parts in double, as these sizes added one FP32 part per 32
// rows in double before they were streamed (m = 10^5, N = 48, relative error of P^T P
// against 64-bit sums: 2.3e-9 so, 2.1e-8 with FP32 chains over a workgroup's rows).
// Past that 512 rows at most (the launches before took a 73rd of m).
template <typename T, int TN>
using RsPart = std::conditional_t<TN <= 4, double, T>;
constexpr int kRsChain = 16;
// Workgroups at m, N: one a CU where that keeps the chains short.
inline int red_stream_groups(int m, int N, int esz) {
  const int nch = (m + kRsRows - 1) / kRsRows;
  int g = kRsGroups;
  if (esz == 4 && N > 64 && nch > kRsChain * g) g = (nch + kRsChain - 1) / kRsChain;
  return nch < g ? nch : g;
}
// Parts of the product, streamed or not.
inline int red_parts(int m, int N, int esz, bool sen) {
  return red_streamed(m, N, esz, sen) ? red_stream_groups(m, N, esz) : (m + kRsRows - 1) / kRsRows;
}
template <typename T, int TN>
constexpr size_t red_stream_lds() {
  return sizeof(T) * 2 * (size_t)(32 * TN) * (kRsRows + 16 / sizeof(T));
}

template <typename T, int TN, bool SEN, int TS>
__global__ __launch_bounds__(kRsThreads) void k_red_stream(int n, int m, int N, int k, int nch,
                                                           const T* Xf, const int32_t* idx,
                                                           const T* hw, const T* y,
                                                           const T* rdiag, const T* eps,
                                                           RsPart<T, TN>* part, int* errw) {
  using C = RsCfg<TN, SEN, TS>;
  using P = RsPart<T, TN>;
  constexpr bool FOLD = sizeof(P) > sizeof(T);
  using V = typename Vec4<T>::type;
  constexpr int KQ = kRsRows / 4, LQ = kRsRows + 16 / (int)sizeof(T), BUF = 32 * TN * LQ;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* qt = (T*)smem_raw;  // two buffers of 32 TN columns (P, then Yt) of LQ
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) bad = 0;
  __syncthreads();
  // ---- the chunk's rows ----
  // The first TB entries of an operator row travel ahead; the rest (k > TB) are
  // read in finish().
  constexpr int RPB = kRsThreads / 32, PASS = kRsRows / RPB;  // rows at once, rows per thread
  constexpr int TB = sizeof(T) == 4 ? 4 : 2;
  const int q = tid & 31, rw = tid >> 5;
  int ci[PASS][TB];  // indices (and weights wn) of the next rows
  T wn[PASS][TB], wc[PASS][TB], xv[PASS][TB][4], ev[PASS][4], yv[PASS], rv[PASS];
  auto load_idx = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PASS; ++u) {
      const int i = ch * kRsRows + u * RPB + rw;
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const bool on = i < m && t < k;
        ci[u][t] = on ? idx[(size_t)i * k + t] : 0;
        wn[u][t] = on ? hw[(size_t)i * k + t] : (T)0;
      }
    }
  };
  auto load_rows = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PASS; ++u) {
      const int i = ch * kRsRows + u * RPB + rw;
      const bool live = i < m;
      yv[u] = live ? y[i] : (T)0;
      rv[u] = live ? rdiag[i] : (T)1;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        ev[u][c] = (live && eps && q + 32 * c < N) ? eps[(size_t)i * N + q + 32 * c] : (T)0;
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        wc[u][t] = wn[u][t];
        if (t < k) {
          int cx = ci[u][t];
          if ((unsigned)cx >= (unsigned)n) {  // (rows past m hold index 0, weight 0)
            if (q == 0) atomicOr(&bad, 2);
            cx = 0;
            wc[u][t] = (T)0;
          }
#pragma unroll
          for (int c = 0; c < 4; ++c)
            xv[u][t][c] = q + 32 * c < N ? Xf[(size_t)cx * N + q + 32 * c] : (T)0;
        }
      }
    }
  };
  auto finish = [&](int ch, T* buf) __attribute__((always_inline)) {
    double h[PASS][4];
#pragma unroll
    for (int u = 0; u < PASS; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        h[u][c] = 0.0;
#pragma unroll
        for (int t = 0; t < TB; ++t)
          if (t < k) h[u][c] += (double)wc[u][t] * (double)xv[u][t][c];
      }
    for (int t = TB; t < k; ++t)
#pragma unroll
      for (int u = 0; u < PASS; ++u) {
        const int i = ch * kRsRows + u * RPB + rw;
        if (i >= m) continue;
        const int cx = idx[(size_t)i * k + t];
        if ((unsigned)cx >= (unsigned)n) {
          if (q == 0) atomicOr(&bad, 2);
          continue;
        }
        const double w = (double)hw[(size_t)i * k + t];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (q + 32 * c < N) h[u][c] += w * (double)Xf[(size_t)cx * N + q + 32 * c];
      }
#pragma unroll
    for (int u = 0; u < PASS; ++u) {
      const int rr = u * RPB + rw;
      const bool live = ch * kRsRows + rr < m;
      const double zb = group_sum<32>((h[u][0] + h[u][1]) + (h[u][2] + h[u][3])) / N;
      double l2 = (double)(N - 1) * (double)rv[u];
      if constexpr (SEN) {
        double ss = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (q + 32 * c < N) ss += (h[u][c] - zb) * (h[u][c] - zb);
        l2 += group_sum<32>(ss);
      }
      const double l = sqrt(l2), yz = (double)yv[u] - zb;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int j = q + 32 * c;
        double pm = 0.0, yt = 0.0;
        if (live && j < N) {
          pm = (h[u][c] - zb) / l;
          yt = (yz + (double)ev[u][c] - (SEN ? h[u][c] - zb : 0.0)) / l;
        }
        if (j < 16 * TN) {
          buf[j * LQ + rr] = (T)pm;
          buf[(16 * TN + j) * LQ + rr] = (T)yt;
        }
      }
    }
  };

  // ---- this wave's tiles (LDS offsets of their columns) ----
  const int lr = lane & 15, lk = lane >> 4;
  const int share = TS > 1 ? blockIdx.y : 0;
  const int t0 = __builtin_amdgcn_readfirstlane(share * kRsWaves + wv) * C::TPW;
  int ao[C::TPW], bo[C::TPW];
#pragma unroll
  for (int i = 0; i < C::TPW; ++i) {
    int t = t0 + i, ta = 0;
    if (t < C::NTL) {
#pragma unroll
      for (int z = 0; z < TN; ++z)  // row ta of the upper triangle starts at ta TN - ta (ta - 1) / 2
        if (t >= (z + 1) * TN - (z + 1) * z / 2) ta = z + 1;
      bo[i] = 16 * (t - ta * TN + ta * (ta - 1) / 2 + ta) * LQ;
      ao[i] = 16 * ta * LQ;
    } else {
      t -= C::NTL;
      ao[i] = 16 * (t / TN) * LQ;
      bo[i] = 16 * (TN + t % TN) * LQ;
    }
  }
  typename Vec4<P>::type acc[C::TPW];
#pragma unroll
  for (int i = 0; i < C::TPW; ++i) acc[i] = {0, 0, 0, 0};
  const int G = gridDim.x;
  int b = 0, ch = blockIdx.x;
  load_idx(ch);
  load_rows(ch);
  load_idx(ch + G);
  for (; ch < nch; ch += G, b ^= 1) {
    // (a wave may still be multiplying the other buffer)
    finish(ch, qt + b * BUF);
    load_rows(ch + G);
    load_idx(ch + 2 * G);
    __syncthreads();
    const T* base = qt + b * BUF + lr * LQ + lk * KQ;
    T av[KQ];
#pragma unroll
    for (int i = 0; i < C::TPW; ++i) {
      if (t0 + i < C::NT) {
        if (i == 0 || ao[i] != ao[i - 1]) vload<KQ>(base + ao[i], av);
        T bv[KQ];
        vload<KQ>(base + bo[i], bv);
        if constexpr (FOLD) {
          V c = V{0, 0, 0, 0};
#pragma unroll
          for (int u = 0; u < KQ; ++u) c = mfma4(av[u], bv[u], c);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][v] += (double)c[v];
        } else {
#pragma unroll
          for (int u = 0; u < KQ; ++u) acc[i] = mfma4(av[u], bv[u], acc[i]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one tile's operands at a time
    }
  }
  __syncthreads();
  if (tid == 0 && share == 0) errw[blockIdx.x] = bad;
  P* out = part + ((size_t)blockIdx.x * C::NT + t0) * 256;
#pragma unroll
  for (int i = 0; i < C::TPW; ++i)
    if (t0 + i < C::NT)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[i * 256 + frag_row<T>(lk, v) * 16 + lr] = acc[i][v];
}

// The sums of k_red_stream's parts (element type P): G (rows of stride LG, both triangles;
// only N x N is written) and B, I added, or, SEN, the update's Wt[b][a] (NP x
// NP, zero outside N x N; zeros to iters0).  A workgroup takes 32 threads of
// 16 consecutive bytes of a tile, eight times: thread row sub adds the parts
// sub, sub + 8, .. in order, then the eight are added in order.
template <typename T, typename P, bool SEN>
__global__ __launch_bounds__(kBlock) void k_red_sum_tiles(int N, int TN, int LG, int S,
                                                          const P* part, double* Gp, double* B,
                                                          T* Wt, int NP, const int* errw, int nerr,
                                                          int* err, int* iters0) {
  constexpr int VU = 16 / (int)sizeof(P);
  __shared__ double red[8][32][VU];
  const int tid = threadIdx.x, x = tid & 31, sub = tid >> 5;
  if (blockIdx.x == 0) {
    if (SEN && iters0)
      for (int e = tid; e < N; e += kBlock) iters0[e] = 0;
    __shared__ int flags;
    if (tid == 0) flags = 0;
    __syncthreads();
    int f = 0;
    for (int e = tid; e < nerr; e += kBlock) f |= errw[e];
    if (f) atomicOr(&flags, f);
    __syncthreads();
    if (tid == 0) *err = flags;
  }
  if (SEN)  // the padding past the tiles
    for (int e = blockIdx.x * kBlock + tid; e < NP * NP; e += gridDim.x * kBlock)
      if (e / NP >= 16 * TN || e % NP >= 16 * TN) Wt[e] = (T)0;
  const int ntl = SEN ? 0 : TN * (TN + 1) / 2, nt = ntl + TN * TN;
  const int e0 = (blockIdx.x * 32 + x) * VU;  // first element (grid: nt * 256 / (32 VU))
  int t = e0 / 256, ti = 0, tj;
  const P* src = part + e0;
  double acc[VU];
#pragma unroll
  for (int v = 0; v < VU; ++v) acc[v] = 0.0;
#pragma unroll 8
  for (int s = sub; s < S; s += 8) {
    P v[VU];
    vload<VU>(src + (size_t)s * nt * 256, v);
#pragma unroll
    for (int u = 0; u < VU; ++u) acc[u] += (double)v[u];
  }
#pragma unroll
  for (int v = 0; v < VU; ++v) red[sub][x][v] = acc[v];
  __syncthreads();
  if (sub != 0) return;
  for (int u = 1; u < 8; ++u)
#pragma unroll
    for (int v = 0; v < VU; ++v) acc[v] += red[u][x][v];
  const bool right = t >= ntl;
  if (right) {
    t -= ntl;
    ti = t / TN;
    tj = t % TN;
  } else {
    while (t >= TN - ti) t -= TN - ti++;
    tj = ti + t;
  }
  const int a = 16 * ti + (e0 % 256) / 16, b0 = 16 * tj + e0 % 16;
#pragma unroll
  for (int v = 0; v < VU; ++v) {
    const int b = b0 + v;
    const double o = acc[v] + (a == b ? 1.0 : 0.0);
    if (SEN) {
      Wt[(size_t)b * NP + a] = (T)((a < N && b < N) ? acc[v] : 0.0);
    } else if (a < N && b < N) {
      if (right) {
        B[(size_t)a * N + b] = o;
      } else {
        Gp[(size_t)a * LG + b] = o;
        if (ti != tj) Gp[(size_t)b * LG + a] = o;
      }
    }
  }
}

// G = I + sum_s part_s[:, :NP] and B = I + sum_s part_s[:, NP:] of k_red_pg's
// parts, restricted to N x N.  Eight lanes share an output: lane q adds the parts q, q + 8, ...
// in order, then a fixed lane tree adds the eight.  G is written as the
// solve keeps it in LDS: NR rows of stride LG, zero outside N x N; B is
// N x N.  Workgroup 0 also folds the gather's error
// words into err.
template <typename T, int NP>
__global__ __launch_bounds__(kBlock) void k_red_sum2(int N, int NR, int LG, int S,
                                                     const T* part, double* Gp, double* B,
                                                     const int* errw, int nerr, int* err) {
  using C = RedCfg<NP>;
  const int tid = threadIdx.x, q = tid & 7;
  if (blockIdx.x == 0) {
    __shared__ int flags;
    if (tid == 0) flags = 0;
    __syncthreads();
    int f = 0;
    for (int e = tid; e < nerr; e += kBlock) f |= errw[e];
    if (f) atomicOr(&flags, f);
    __syncthreads();
    if (tid == 0) *err = flags;
  }
  const int o = blockIdx.x * (kBlock / 8) + tid / 8, ng = NR * LG, total = ng + N * N;
  const bool right = o >= ng;
  int a = 0, b = 0;
  bool live = o < total;
  if (live) {
    if (!right) {
      a = o / LG;
      b = o - a * LG;
      live = a < N && b < N;
    } else {
      a = (o - ng) / N;
      b = (o - ng) - a * N;
    }
  }
  double acc = 0.0;
  if (live) {
    const T* src = part + (size_t)a * C::QW + (right ? NP : 0) + b;
    const size_t stride = (size_t)NP * C::QW;
#pragma unroll 4
    for (int s = q; s < S; s += 8) acc += (double)src[s * stride];
  }
  acc = group_sum<8>(acc);
  if (q == 0 && o < total) {
    if (live && a == b) acc += 1.0;
    if (right)
      B[o - ng] = acc;
    else
      Gp[o] = acc;
  }
}

// sEnKF: Zhat^T diag(...)^{-1} (Y - Z) = sum_s part_s[:, NP:] restricted to
// N x N, written transposed in the update's element type as k_red_update
// takes W' - I: Wt[b][a] (NP x NP, zero outside N x N).  Eight lanes share an
// output as in k_red_sum2; workgroup 0 folds the gather's error words and
// zeros the N iteration counts (iters0, if given: no CG runs).
template <typename T, int NP>
__global__ __launch_bounds__(kBlock) void k_senkf_sum(int N, int S, const T* part, T* Wt,
                                                      const int* errw, int nerr, int* err,
                                                      int* iters0) {
  using C = RedCfg<NP>;
  const int tid = threadIdx.x, q = tid & 7;
  if (blockIdx.x == 0) {
    if (iters0)
      for (int e = tid; e < N; e += kBlock) iters0[e] = 0;
    __shared__ int flags;
    if (tid == 0) flags = 0;
    __syncthreads();
    int f = 0;
    for (int e = tid; e < nerr; e += kBlock) f |= errw[e];
    if (f) atomicOr(&flags, f);
    __syncthreads();
    if (tid == 0) *err = flags;
  }
  const int o = blockIdx.x * (kBlock / 8) + tid / 8;  // all eight lanes of a group share o
  if (o >= NP * NP) return;
  const int b = o / NP, a = o - b * NP;
  double acc = 0.0;
  if (a < N && b < N) {
    const T* src = part + (size_t)a * C::QW + NP + b;
    const size_t stride = (size_t)NP * C::QW;
#pragma unroll 4
    for (int s = q; s < S; s += 8) acc += (double)src[s * stride];
  }
  acc = group_sum<8>(acc);
  if (q == 0) Wt[o] = (T)acc;
}

// CGD-EnKF-Reduced solve for N <= 64 RPL: textbook CG on G w = b_j from
// w = 0 (Lemma 1: at most N steps in exact arithmetic), one workgroup per
// column.  G comes as the sum launch lays it out (stride LG = 64 RPL; only N x
// N is read); each wave keeps a quarter of its rows in
// registers (reading G from LDS every step cost 0.43 us a step at N = 128).
// Each wave carries the whole recurrence (lane l holds rows l + 64 u of w,
// r, p, q), the same values in every wave, but forms only a quarter of
// q = G p: the rows of G from LG/4 wv on, with its own copy of p in LDS.  The four partial q meet
// in LDS (two buffers, alternate steps) behind one barrier per step and
// every wave adds them in the same order, so all waves take the same
// decisions.  Writes W (FP64, row-major) and Wt = (W - I)^T in the update's
// element type (NP x NP, zero outside N x N); workgroups j >= N only clear
// their row of Wt.
template <typename T, int RPL>
__global__ __launch_bounds__(kBlock) void k_small_cg_w(int N, int NP, const double* Gp,
                                                       const double* B, double* W, T* Wt,
                                                       int* iters, int* iters2, int* status,
                                                       double tol, int maxit) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int LG = 64 * RPL, NW = kBlock / 64, QR = LG / NW;
  static_assert(QR % 16 == 0, "rows per wave");
  double* ps = (double*)smem_raw;             // NW x LG
  double* qp = ps + (size_t)NW * LG;          // 2 x NW x LG
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = blockIdx.x;
  if (j >= N) {
    for (int e = tid; e < NP; e += kBlock) Wt[(size_t)j * NP + e] = (T)0;
    return;
  }
  // This wave's QR rows of G (G is symmetric: row l, column i = lane + 64 u),
  // kept in registers for the whole solve (QR x RPL doubles per lane), so
  // that a step reads no G from LDS.
  double gr[QR][RPL];
#pragma unroll
  for (int t = 0; t < QR; ++t)
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const int l = wv * QR + t, i = lane + 64 * u;
      gr[t][u] = l < N && i < N ? Gp[(size_t)l * LG + i] : 0.0;
    }
  double x[RPL], r[RPL], p[RPL];
  double part = 0.0;
#pragma unroll
  for (int u = 0; u < RPL; ++u) {
    const int i = lane + 64 * u;
    const double b = i < N ? B[(size_t)i * N + j] : 0.0;
    x[u] = 0.0;
    r[u] = b;
    p[u] = b;
    part += b * b;
  }
  double rho = wave_sum(part);
  const double thr = tol * sqrt(rho);
  double* myp = ps + wv * LG;
  int it = 0, buf = 0;
  bool nonfinite = false;
  while (sqrt(rho) > thr && it < maxit && rho > 0.0) {
#pragma unroll
    for (int u = 0; u < RPL; ++u) myp[lane + 64 * u] = p[u];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // this wave's quarter of q = G p, four accumulation chains
    double qa[4][RPL];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int u = 0; u < RPL; ++u) qa[c][u] = 0.0;
#pragma unroll
    for (int c = 0; c < QR / 16; ++c) {
      const int l0 = wv * QR + 16 * c;
      v2d pv[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) pv[t] = *reinterpret_cast<const v2d*>(myp + l0 + 2 * t);
#pragma unroll
      for (int t = 0; t < 16; ++t)
#pragma unroll
        for (int u = 0; u < RPL; ++u) qa[t & 3][u] += gr[16 * c + t][u] * pv[t >> 1][t & 1];
    }
    double* qw = qp + (size_t)(buf * NW + wv) * LG;
#pragma unroll
    for (int u = 0; u < RPL; ++u)
      qw[lane + 64 * u] = (qa[0][u] + qa[1][u]) + (qa[2][u] + qa[3][u]);
    __syncthreads();
    const double* qb = qp + (size_t)buf * NW * LG;
    buf ^= 1;
    double q[RPL];
    part = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const int i = lane + 64 * u;
      q[u] = (qb[i] + qb[LG + i]) + (qb[2 * LG + i] + qb[3 * LG + i]);
      part += p[u] * q[u];
    }
    const double alpha = rho / wave_sum(part);
    part = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      x[u] += alpha * p[u];
      r[u] -= alpha * q[u];
      part += r[u] * r[u];
    }
    const double rho_new = wave_sum(part);
    const double beta = rho_new / rho;
#pragma unroll
    for (int u = 0; u < RPL; ++u) p[u] = r[u] + beta * p[u];
    rho = rho_new;
    ++it;
    // alpha and beta are the same in every lane and wave, so the exit is uniform
    if (!isfinite(alpha) || !isfinite(beta)) {
      nonfinite = true;
      break;
    }
  }
  if (wv != 0) return;
#pragma unroll
  for (int u = 0; u < RPL; ++u) {
    const int i = lane + 64 * u;
    if (i < N) W[(size_t)i * N + j] = x[u];
    if (i < NP) Wt[(size_t)j * NP + i] = (T)(i < N ? x[u] - (i == j ? 1.0 : 0.0) : 0.0);
  }
  if (lane == 0) {
    iters[j] = it;
    if (iters2) iters2[j] = it;
    status[j] = small_cg_status(nonfinite, rho, thr);
  }
}

// X_a = X_f + X_f (W - I) on the MFMA with W'^T = Wt read as prepared by the
// solve; RB-row tiles so that small n still spreads over the chip.
template <typename T, int NP, int RB>
__global__ __launch_bounds__(kBlock) void k_red_update(int n, int N, const T* Xf, T* Xa,
                                                       const T* Wtg) {
  using U = UCfg<T, NP, RB>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* Wt = (T*)smem_raw;
  T* As = Wt + (size_t)NP * U::LD;
  double* mean = (double*)(As + (size_t)U::RBX * U::LD);
  // W'^T once per workgroup (16-byte loads, all in flight at once)
  constexpr int VW = 16 / (int)sizeof(T), NWL = NP * NP / VW / kBlock;
  static_assert(NWL * VW * kBlock == NP * NP, "W loads");
  const int tid = threadIdx.x;
  T wl[NWL][VW];
#pragma unroll
  for (int u = 0; u < NWL; ++u) {
    const int e = u * kBlock + tid, row = e / (NP / VW), c = (e - row * (NP / VW)) * VW;
    vload<VW>(Wtg + (size_t)row * NP + c, wl[u]);
  }
#pragma unroll
  for (int u = 0; u < NWL; ++u) {
    const int e = u * kBlock + tid, row = e / (NP / VW), c = (e - row * (NP / VW)) * VW;
#pragma unroll
    for (int v = 0; v < VW; ++v) Wt[row * U::LD + c + v] = wl[u][v];
  }
  update_tiles_stream<T, NP, kBlock, RB>(n, N, Xf, Xa, 1, As, As, Wt, mean);
}

// ---------------------------------------------------------------------------
// Reduced mode and sEnKF for N > 128, in FP64 whatever T is: NP = N rounded up
// to 64, Q (mpad x 2NP, as above, in double) through memory, the product on
// the FP64 MFMA in 64 x 64 tiles over row chunks.  Past kRedPanel rows Q holds one
// panel of rows at a time, so that the workspace stops growing there.  (One workgroup per row
// block with a scalar FP64 sum per output, and a serial sum over up to 1024
// N x 2N parts, took 277 + 88 us at m = 5003, N = 200.)
// ---------------------------------------------------------------------------

// Row i of Q (in row i - p0 of the panel that starts at p0), one wave per row.  HX is
// kept in the row's left half until its mean is known.  errw: an error word per
// workgroup, kept over the panels; SEN: the sEnKF's row scale.
template <typename T, bool SEN>
__global__ __launch_bounds__(kBlock) void k_red_prep_wide(int n, int m, int p0, int N, int NP,
                                                          int k, const T* Xf, const int32_t* idx,
                                                          const T* hw, const T* y, const T* rdiag,
                                                          const T* eps, double* Q, int* errw) {
  __shared__ int bad;
  const int lane = threadIdx.x & 63, row = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int i = p0 + row;
  if (threadIdx.x == 0) bad = p0 > 0 ? errw[blockIdx.x] : 0;
  __syncthreads();
  double* qr = Q + (size_t)row * 2 * NP;
  const bool live = i < m;
  constexpr int U = 4;
  double sum = 0.0;
  for (int j0 = lane; j0 < NP; j0 += 64 * U) {
    double h[U];
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = 0.0;
    if (live)
      for (int t = 0; t < k; ++t) {
        const int c = idx[(size_t)i * k + t];
        if ((unsigned)c >= (unsigned)n) {
          if (lane == 0) atomicOr(&bad, 2);
          continue;
        }
        const double w = (double)hw[(size_t)i * k + t];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (j0 + 64 * u < N) h[u] += w * (double)Xf[(size_t)c * N + j0 + 64 * u];
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + 64 * u < NP) {
        qr[j0 + 64 * u] = h[u];
        sum += h[u];
      }
  }
  const double zb = wave_sum(sum) / N;
  double l2 = live ? (double)(N - 1) * (double)rdiag[i] : 1.0;
  if constexpr (SEN) {
    double ss = 0.0;
    for (int j = lane; j < N; j += 64) ss += (qr[j] - zb) * (qr[j] - zb);
    l2 += wave_sum(ss);
  }
  const double l = sqrt(l2), yv = live ? (double)y[i] : 0.0;
  for (int j = lane; j < NP; j += 64) {
    const bool on = live && j < N;
    const double h = qr[j];
    double yt = yv - (SEN ? h : zb);
    if (on && eps) yt += (double)eps[(size_t)i * N + j];
    qr[j] = on ? (h - zb) / l : 0.0;
    qr[NP + j] = on ? yt / l : 0.0;
  }
  __syncthreads();
  if (threadIdx.x == 0) errw[blockIdx.x] = bad;
}

// part[s] = Q[rows of chunk s, :NP]^T Q[rows of chunk s, :] of a panel of mpad rows
// (add: onto the panels before it), tiles t0 .. of the tile list (all of the right
// half, the left half's lower tiles skipped).  All tiles of a chunk run on one XCD
// (workgroup w runs on XCD w mod 8), whose L2 then serves the chunk's rows to
// every tile after the first.
__global__ __launch_bounds__(kBlock) void k_red_gemm_wide(int NP, int KC, int mpad, int S, int t0,
                                                          int ntile, int add, const double* Q,
                                                          double* part) {
  constexpr int MB = 2, HS = 32;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  const int TT = NP / 64, NTG = TT * (TT + 1) / 2, slot = blockIdx.x / 8;
  const int chunk = (int)(blockIdx.x % 8) + 8 * (slot / ntile);
  if (chunk >= S) return;
  int t = t0 + slot % ntile, ta = 0, tb;
  if (t < NTG) {
    while (t >= TT - ta) t -= TT - ta++;
    tb = ta + t;
  } else {
    t -= NTG;
    ta = t / TT;
    tb = TT + t % TT;
  }
  const int ca = ta * 64 + (wv >> 1) * HS + lr, cb = tb * 64 + (wv & 1) * HS + lr;
  const int r0 = chunk * KC, r1 = min(mpad, r0 + KC);
  if (r0 >= r1) return;  // (a last, shorter panel)
  const size_t QW = 2 * (size_t)NP;
  double* out = part + (size_t)chunk * NP * QW;
  auto at = [&](int x, int z, int i) {
    return (size_t)(ca - lr + 16 * x + frag_row<double>(lk, i)) * QW + cb + 16 * z;
  };
  v4d acc[MB][MB];
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int z = 0; z < MB; ++z)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[x][z][i] = add ? out[at(x, z, i)] : 0.0;
  double an[4][MB], bn[4][MB];
  auto load = [&](int r) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double* row = Q + (size_t)(r + 4 * u + lk) * QW;
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        an[u][x] = row[ca + 16 * x];
        bn[u][x] = row[cb + 16 * x];
      }
    }
  };
  load(r0);
  for (int r = r0; r < r1; r += 16) {
    double ac[4][MB], bc[4][MB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        ac[u][x] = an[u][x];
        bc[u][x] = bn[u][x];
      }
    if (r + 16 < r1) load(r + 16);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int z = 0; z < MB; ++z) acc[x][z] = mfma4(ac[u][x], bc[u][z], acc[x][z]);
  }
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int z = 0; z < MB; ++z)
#pragma unroll
      for (int i = 0; i < 4; ++i) out[at(x, z, i)] = acc[x][z][i];
}

// G = I + sum_s part_s[:, :NP] (from its upper tiles; stride LG, rows and
// columns < LG) and B = dadd I + sum_s part_s[:, NP:] (N x N), parts in order.
// left = 0: B only.  Workgroup 0 folds the gather's error words into err.
__global__ __launch_bounds__(kBlock) void k_red_sum_wide(int N, int NP, int LG, int S, int left,
                                                         double dadd, const double* part,
                                                         double* G, double* B, const int* errw,
                                                         int nerr, int* err) {
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    __shared__ int flags;
    if (tid == 0) flags = 0;
    __syncthreads();
    int f = 0;
    for (int e = tid; e < nerr; e += kBlock) f |= errw[e];
    if (f) atomicOr(&flags, f);
    __syncthreads();
    if (tid == 0) *err = flags;
  }
  const int W = left ? 2 * NP : NP, o = blockIdx.x * kBlock + tid;
  if (o >= NP * W) return;
  const int a = o / W, b = o - a * W + (left ? 0 : NP);
  const bool right = b >= NP;
  const int bb = right ? b - NP : b;
  if (right ? (a >= N || bb >= N) : (a / 64 > bb / 64)) return;
  const size_t stride = (size_t)NP * 2 * NP;
  const double* src = part + (size_t)a * 2 * NP + b;
  double acc = 0.0;
#pragma unroll 8
  for (int s = 0; s < S; ++s) acc += src[s * stride];
  if (right) {
    B[(size_t)a * N + bb] = acc + (a == bb ? dadd : 0.0);
  } else if (a < LG && bb < LG) {
    if (a == bb && a < N) acc += 1.0;
    G[(size_t)a * LG + bb] = acc;
    if (a / 64 < bb / 64) G[(size_t)bb * LG + a] = acc;
  }
}

// The column CG of k_small_cg for 128 < N <= 256 with G on chip (stride LG = 64
// RPL, zero outside N x N): eight waves, each with QR rows of G (8 QR >= N), RR
// of them in registers and the rest in LDS, since 512 KiB of G at LG =
// 256 fit neither alone.  Every wave carries the whole recurrence and forms
// its rows' part of q = G p (see k_small_cg_w); the eight parts meet in LDS.
// Reading G from L2 every step took 378 us for 200 columns, 16 steps; this 38 us.
// (RR = 24: with 26 rows a wave, N <= 208, nothing spills; with 28 and 32 it is 8 and 11
// VGPRs, and with 32 the LDS holds no more rows.)
template <int RPL, int QRows>
struct SmallCgX {
  static constexpr int LG = 64 * RPL, NW = 8, QR = QRows, RR = 24, RL = QR - RR;
  static constexpr size_t lds = sizeof(double) * ((size_t)NW * RL * LG + NW * LG + NW * QR + LG);
};
template <int RPL, int QRows>
__global__ __launch_bounds__(512) void k_small_cg_x(int N, const double* Gp, const double* B,
                                                    double* W, int* iters, int* iters2,
                                                    int* status, double tol, int maxit) {
  using C = SmallCgX<RPL, QRows>;
  constexpr int LG = C::LG, NW = C::NW, QR = C::QR, RR = C::RR, RL = C::RL;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* gl = (double*)smem_raw;         // NW x RL x LG
  double* qp = gl + (size_t)NW * RL * LG; // NW x LG
  double* ps = qp + NW * LG;              // NW x QR
  double* xs = ps + NW * QR;              // LG: the iterate, kept by wave 0 (registers are short)
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = blockIdx.x;
  const int l0 = wv * QR;
  double gr[RR][RPL];
#pragma unroll
  for (int t = 0; t < RR; ++t)
#pragma unroll
    for (int u = 0; u < RPL; ++u) gr[t][u] = Gp[(size_t)(l0 + t) * LG + lane + 64 * u];
  double* myg = gl + (size_t)wv * RL * LG;
#pragma unroll
  for (int t = 0; t < RL; ++t)
#pragma unroll
    for (int u = 0; u < RPL; ++u)
      myg[t * LG + lane + 64 * u] = Gp[(size_t)(l0 + RR + t) * LG + lane + 64 * u];
  double r[RPL], p[RPL];
  double part = 0.0;
#pragma unroll
  for (int u = 0; u < RPL; ++u) {
    const int i = lane + 64 * u;
    const double b = i < N ? B[(size_t)i * N + j] : 0.0;
    if (wv == 0) xs[i] = 0.0;
    r[u] = b;
    p[u] = b;
    part += b * b;
  }
  double rho = wave_sum(part);
  const double thr = tol * sqrt(rho);
  double* myp = ps + wv * QR;
  int it = 0;
  bool nonfinite = false;
  while (sqrt(rho) > thr && it < maxit && rho > 0.0) {
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const int i = lane + 64 * u - l0;
      if (i >= 0 && i < QR) myp[i] = p[u];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double qa[RPL];
#pragma unroll
    for (int u = 0; u < RPL; ++u) qa[u] = 0.0;
#pragma unroll
    for (int t = 0; t < QR; t += 2) {
      const v2d pv = *reinterpret_cast<const v2d*>(myp + t);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int u = 0; u < RPL; ++u) {
          double g;
          if constexpr (RL > 0) {
            g = t + c < RR ? gr[t + c < RR ? t + c : 0][u]
                           : myg[(t + c - RR) * LG + lane + 64 * u];
          } else {
            g = gr[t + c][u];
          }
          qa[u] += g * pv[c];
        }
    }
    __syncthreads();  // the previous step's sums are read
    double* qw = qp + (size_t)wv * LG;
#pragma unroll
    for (int u = 0; u < RPL; ++u) qw[lane + 64 * u] = qa[u];
    __syncthreads();
    double q[RPL];
    part = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const double* qb = qp + lane + 64 * u;
      double v = qb[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += qb[(size_t)w * LG];
      q[u] = v;
      part += p[u] * v;
    }
    const double alpha = rho / wave_sum(part);
    part = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      if (wv == 0) xs[lane + 64 * u] += alpha * p[u];
      r[u] -= alpha * q[u];
      part += r[u] * r[u];
    }
    const double rho_new = wave_sum(part);
    const double beta = rho_new / rho;
#pragma unroll
    for (int u = 0; u < RPL; ++u) p[u] = r[u] + beta * p[u];
    rho = rho_new;
    ++it;
    // the same bits in every lane and wave, so the exit is uniform
    if (!isfinite(alpha) || !isfinite(beta)) {
      nonfinite = true;
      break;
    }
  }
  if (wv != 0) return;
#pragma unroll
  for (int u = 0; u < RPL; ++u) {
    const int i = lane + 64 * u;
    if (i < N) W[(size_t)i * N + j] = xs[i];
  }
  if (lane == 0) {
    iters[j] = it;
    if (iters2) iters2[j] = it;
    status[j] = small_cg_status(nonfinite, rho, thr);
  }
}

template <int RPL, int QR>
hipError_t launch_small_cg_x(int N, const double* G, const double* B, double* W, int* iters,
                             int* iters2, int* status, double tol, int maxit, hipStream_t s) {
  constexpr size_t lds = SmallCgX<RPL, QR>::lds;
  const hipError_t e = hipFuncSetAttribute((const void*)k_small_cg_x<RPL, QR>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_small_cg_x<RPL, QR>), dim3(N), dim3(512), lds, s, N, G, B, W, iters, iters2,
                     status, tol, maxit);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_validate(int n, int m, int N, int k, const T* Xf,
                                                     const int32_t* idx, const T* hw, const T* y,
                                                     const T* rdiag, const T* eps, const T* z0,
                                                     int* flags) {
  const size_t stride = (size_t)gridDim.x * kBlock;
  const size_t t0 = (size_t)blockIdx.x * kBlock + threadIdx.x;
  int f = 0;
  for (size_t e = t0; e < (size_t)n * N; e += stride)
    if (!isfinite((double)Xf[e])) f |= VF_NONFINITE;
  for (size_t e = t0; e < (size_t)m * k; e += stride) {
    if (idx[e] < 0 || idx[e] >= n) f |= VF_INDEX;
    if (!isfinite((double)hw[e])) f |= VF_NONFINITE;
  }
  for (size_t e = t0; e < (size_t)m; e += stride) {
    if (!isfinite((double)y[e]) || !isfinite((double)rdiag[e])) f |= VF_NONFINITE;
    if (!(rdiag[e] > (T)0)) f |= VF_NONPOS_R;
  }
  if (eps)
    for (size_t e = t0; e < (size_t)m * N; e += stride)
      if (!isfinite((double)eps[e])) f |= VF_NONFINITE;
  if (z0)
    for (size_t e = t0; e < (size_t)m * N; e += stride)
      if (!isfinite((double)z0[e])) f |= VF_NONFINITE;
  if (f) atomicOr(flags, f);
}

inline int update_rows(int N) {
  int r = (int)((32 * 1024) / (sizeof(double) * (size_t)N + 8));
  if (r > 64) r = 64;
  return r < 1 ? 1 : r;
}

}  // namespace

template <typename T>
hipError_t launch_update(int n, int N, const T* Xf, T* Xa, const double* Wd, int mode,
                         hipStream_t s, const int* skip) {
  if (N <= 128 && update_rows_ok(n, N, Xf, Xa))
    return launch_update_rows<T, false>(n, N, 0, Xf, Xa, Wd, nullptr, mode, skip, s);
  if (N <= 16) return launch_update_mfma<T, 16>(n, N, Xf, Xa, Wd, mode, skip, s);
  if (N <= 32) return launch_update_mfma<T, 32>(n, N, Xf, Xa, Wd, mode, skip, s);
  if (N <= 64) return launch_update_mfma<T, 64>(n, N, Xf, Xa, Wd, mode, skip, s);
  if constexpr (sizeof(T) == 4)
    if (N <= 128) return launch_update_mfma<T, 128>(n, N, Xf, Xa, Wd, mode, skip, s);
  // larger ensembles: 32 rows a workgroup while they fit its LDS, else 16, else
  // (N past 1000) one double FMA chain per element
  if (update_wide_lds<T>(N, 2) <= kUpdWideLds)
    return launch_update_wide<T, 2>(n, N, Xf, Xa, Wd, mode, skip, s);
  if (update_wide_lds<T>(N, 1) <= kUpdWideLds)
    return launch_update_wide<T, 1>(n, N, Xf, Xa, Wd, mode, skip, s);
  const int RBX = update_rows(N);
  const size_t sh = sizeof(double) * ((size_t)RBX * N + RBX);
  hipLaunchKernelGGL(k_update<T>, dim3((n + RBX - 1) / RBX), dim3(kBlock), sh, s, n, N, RBX, Xf,
                     Xa, Wd, mode, skip);
  return hipGetLastError();
}

int reduced_shape(int m, int N, int* NP, int* mpad) {
  if (N < 2 || N > 128 || m < 1 || m > (1 << 30)) return 0;
  static_assert(kRedFusedRows == kRsRows, "one chunk height");
  const int nch = (m + kRsRows - 1) / kRsRows;
  *NP = N <= 32 ? 32 : N <= 64 ? 64 : 128;
  *mpad = nch * kRsRows;
  return 1;
}

// A part holds all of NP x 2NP from k_red_pg, else its 16 x 16 tiles (RsPart).
size_t reduced_parts_bytes(int m, int N, int esz) {
  size_t most = 0;
  for (const bool sen : {false, true}) {
    const size_t tn = red_stream_tiles(N), np = N <= 32 ? 32 : 64;
    const size_t part = red_streamed(m, N, esz, sen)
                            ? (tn * (tn + 1) / 2 + tn * tn) * 256 * (tn <= 4 ? sizeof(double) : esz)
                            : np * 2 * np * esz;
    most = std::max(most, part * red_parts(m, N, esz, sen));
  }
  return most;
}

void reduced_wide_shape(int m, int N, int* NP, int* mpad, int* KC, int* S) {
  const int np = (N + 63) / 64 * 64, TT = np / 64, tiles = TT * (TT + 1) / 2 + TT * TT;
  const long mp = ((long)(m < kRedPanel ? m : kRedPanel) + 31) / 32 * 32, blocks = mp / 32;
  // about 512 workgroups, in whole rounds over the eight XCDs, chunks of at
  // least 64 rows
  long sc = (512 / tiles + 7) / 8 * 8;
  const long smax = (mp + 63) / 64;
  if (sc > smax) sc = smax;
  if (sc < 1) sc = 1;
  const long kc = (blocks + sc - 1) / sc * 32;
  *NP = np;
  *mpad = (int)mp;
  *KC = (int)kc;
  *S = (int)((mp + kc - 1) / kc);
}

namespace {

template <typename T, int NP, int RB>
hipError_t launch_red_update(int n, int N, const T* Xf, T* Xa, const T* Wt, hipStream_t s) {
  using U = UCfg<T, NP, RB>;
  hipError_t e = hipFuncSetAttribute((const void*)k_red_update<T, NP, RB>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)U::lds);
  if (e != hipSuccess) return e;
  // persistent: as many workgroups as run at once (each loads W once), at
  // most one per tile
  static int resident = 0;
  if (resident == 0) {
    int dev = 0, cus = 0, per = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
        hipSuccess)
      return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_red_update<T, NP, RB>, kBlock,
                                                          U::lds)) != hipSuccess)
      return e;
    resident = per * cus > 0 ? per * cus : 1;
  }
  const int tiles = (n + RB - 1) / RB;
  const int grid = tiles < resident ? tiles : resident;
  hipLaunchKernelGGL((k_red_update<T, NP, RB>), dim3(grid), dim3(kBlock), U::lds, s, n, N, Xf,
                     Xa, Wt);
  return hipGetLastError();
}

// The tallest row tile that fits the LDS and still gives every CU a workgroup.
template <typename T, int NP>
hipError_t launch_red_update_np(int n, int N, const T* Xf, T* Xa, const T* Wt, hipStream_t s) {
  if (update_rows_ok(n, N, Xf, (const T*)Xa))
    return launch_update_rows<T, true>(n, N, NP, Xf, Xa, nullptr, Wt, 1, nullptr, s);
  constexpr size_t lmax = 160 * 1024;
  if constexpr (UCfg<T, NP, 64>::lds <= lmax)
    if (n >= 64 * 256) return launch_red_update<T, NP, 64>(n, N, Xf, Xa, Wt, s);
  if constexpr (UCfg<T, NP, 32>::lds <= lmax)
    if (n >= 32 * 256) return launch_red_update<T, NP, 32>(n, N, Xf, Xa, Wt, s);
  static_assert(UCfg<T, NP, 16>::lds <= lmax, "update tile");
  return launch_red_update<T, NP, 16>(n, N, Xf, Xa, Wt, s);
}

// The two launches of a streamed product: the parts, then their sums (B null: the
// sEnKF's, into Wt).
template <typename T, int TN, bool SEN, int TS>
hipError_t launch_red_stream_tn(int n, int m, int N, int k, const T* Xg, const int32_t* idx,
                                const T* hw, const T* y, const T* rdiag, const T* eps, void* ws,
                                const Layout& L, int* iters0, hipStream_t s) {
  using P = RsPart<T, TN>;
  using C = RsCfg<TN, SEN, TS>;
  const int S = red_parts(m, N, sizeof(T), SEN);
  unsigned char* base = (unsigned char*)ws;
  P* part = (P*)(base + L.rpart);
  int* errw = (int*)(base + L.rerr);
  constexpr size_t lds = red_stream_lds<T, TN>();
  hipError_t e = hipFuncSetAttribute((const void*)k_red_stream<T, TN, SEN, TS>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_red_stream<T, TN, SEN, TS>), dim3(S, TS), dim3(kRsThreads), lds, s, n, m,
                     N, k, (m + kRsRows - 1) / kRsRows, Xg, idx, hw, y, rdiag, eps, part, errw);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL((k_red_sum_tiles<T, P, SEN>), dim3(C::NT * 8 * sizeof(P) / 16), dim3(kBlock),
                     0, s, N, TN, L.rNP < 64 ? 64 : L.rNP, S, (const P*)part,
                     SEN ? nullptr : (double*)(base + L.rG), SEN ? nullptr : (double*)(base + L.rB),
                     SEN ? (T*)(base + L.rWt) : nullptr, L.rNP, (const int*)errw, S,
                     (int*)(base + L.err), iters0);
  return hipGetLastError();
}
template <typename T, bool SEN>
hipError_t launch_red_stream(int n, int m, int N, int k, const T* Xg, const int32_t* idx,
                             const T* hw, const T* y, const T* rdiag, const T* eps, void* ws,
                             const Layout& L, int* iters0, hipStream_t s) {
  auto one = [&](auto tn) {
    constexpr int TN = decltype(tn)::value;
    if constexpr (TN > 4)
      if (red_stream_split(m, N))
        return launch_red_stream_tn<T, TN, SEN, kRsSplit>(n, m, N, k, Xg, idx, hw, y, rdiag, eps,
                                                          ws, L, iters0, s);
    return launch_red_stream_tn<T, TN, SEN, 1>(n, m, N, k, Xg, idx, hw, y, rdiag, eps, ws, L,
                                               iters0, s);
  };
  switch (red_stream_tiles(N)) {
    case 2: return one(std::integral_constant<int, 2>{});
    case 3: return one(std::integral_constant<int, 3>{});
    case 4: return one(std::integral_constant<int, 4>{});
    case 5: return one(std::integral_constant<int, 5>{});
    case 6: return one(std::integral_constant<int, 6>{});
    case 7: return one(std::integral_constant<int, 7>{});
    default: return one(std::integral_constant<int, 8>{});
  }
}

template <typename T, int NP>
hipError_t launch_reduced_mfma(int n, int m, int N, int k, const T* Xf, T* Xa, const T* Xg, int ng,
                               const int32_t* idx, const T* hw, const T* y, const T* rdiag,
                               const T* eps, double tol, int maxit, void* ws, const Layout& L,
                               int* iters_out, hipStream_t s) {
  unsigned char* base = (unsigned char*)ws;
  T* part = (T*)(base + L.rpart);
  double* Gp = (double*)(base + L.rG);
  double* B = (double*)(base + L.rB);
  double* Wd = (double*)(base + L.Wd);
  T* Wt = (T*)(base + L.rWt);
  int* iters = (int*)(base + L.riters);
  int* stat = (int*)(base + L.rstat);
  int* err = (int*)(base + L.err);
  int* errw = (int*)(base + L.rerr);
  const int LG = NP < 64 ? 64 : NP, RPL = LG / 64, NR = LG;
  hipError_t e;
  if (red_streamed(m, N, sizeof(T), false)) {
    if ((e = launch_red_stream<T, false>(ng, m, N, k, Xg, idx, hw, y, rdiag, eps, ws, L, nullptr,
                                         s)) != hipSuccess)
      return e;
  } else if constexpr (NP <= 64) {
    const int S = red_parts(m, N, sizeof(T), false);
    hipLaunchKernelGGL((k_red_pg<T, NP, false>), dim3(S), dim3(kBlock), 0, s, ng, m, N, k, Xg,
                       idx, hw, y, rdiag, eps, part, errw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int nsum = NR * LG + N * N, per = kBlock / 8;
    hipLaunchKernelGGL((k_red_sum2<T, NP>), dim3((nsum + per - 1) / per), dim3(kBlock), 0, s, N,
                       NR, LG, S, (const T*)part, Gp, B, (const int*)errw, S, err);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t lds = sizeof(double) * (3 * (kBlock / 64) * (size_t)LG);
  if (RPL == 1) {
    if ((e = hipFuncSetAttribute((const void*)k_small_cg_w<T, 1>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
        hipSuccess)
      return e;
    hipLaunchKernelGGL((k_small_cg_w<T, 1>), dim3(NP), dim3(kBlock), lds, s, N, NP,
                       (const double*)Gp, (const double*)B, Wd, Wt, iters, iters_out, stat, tol,
                       maxit);
  } else {
    if ((e = hipFuncSetAttribute((const void*)k_small_cg_w<T, 2>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
        hipSuccess)
      return e;
    hipLaunchKernelGGL((k_small_cg_w<T, 2>), dim3(NP), dim3(kBlock), lds, s, N, NP,
                       (const double*)Gp, (const double*)B, Wd, Wt, iters, iters_out, stat, tol,
                       maxit);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_red_update_np<T, NP>(n, N, Xf, Xa, Wt, s);
}

}  // namespace

namespace {
// N > 128: Q, its product's parts and their sums (G and B; B only for SEN).
template <typename T, bool SEN>
hipError_t red_wide_product(int ng, int m, int N, int k, const T* Xg, const int32_t* idx,
                            const T* hw, const T* y, const T* rdiag, const T* eps, void* ws,
                            const Layout& L, hipStream_t s) {
  unsigned char* base = (unsigned char*)ws;
  double* Q = (double*)(base + L.rQ);
  double* part = (double*)(base + L.rpart);
  int* errw = (int*)(base + L.rerr);
  const int NP = L.rWNP, nprep = L.rmpad / (kBlock / 64), TT = NP / 64, NTG = TT * (TT + 1) / 2;
  const int t0 = SEN ? NTG : 0, ntile = NTG + TT * TT - t0;
  hipError_t e;
  for (long at = 0; at < m; at += kRedPanel) {
    const int p0 = (int)at, rows = m - p0 < kRedPanel ? m - p0 : kRedPanel;
    const int mpad = (rows + 31) / 32 * 32;
    const int KC = p0 == 0 ? L.rKC : (mpad / 32 + L.rS - 1) / L.rS * 32;  // all parts busy
    hipLaunchKernelGGL((k_red_prep_wide<T, SEN>), dim3(mpad / (kBlock / 64)), dim3(kBlock), 0, s,
                       ng, m, p0, N, NP, k, Xg, idx, hw, y, rdiag, eps, Q, errw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_red_gemm_wide, dim3(8 * ntile * ((L.rS + 7) / 8)), dim3(kBlock), 0, s,
                       NP, KC, mpad, L.rS, t0, ntile, p0 > 0 ? 1 : 0, (const double*)Q, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int W = SEN ? NP : 2 * NP;
  hipLaunchKernelGGL(k_red_sum_wide, dim3((NP * W + kBlock - 1) / kBlock), dim3(kBlock), 0, s, N,
                     NP, L.rLG, L.rS, SEN ? 0 : 1, SEN ? 0.0 : 1.0, (const double*)part,
                     (double*)(base + L.rG), (double*)(base + L.rB), (const int*)errw, nprep,
                     (int*)(base + L.err));
  return hipGetLastError();
}
}  // namespace

template <typename T>
hipError_t launch_reduced(int n, int m, int N, int k, const T* Xf, T* Xa, const T* Xg, int ng,
                          const int32_t* idx, const T* hw, const T* y, const T* rdiag,
                          const T* eps, double tol, int maxit, void* ws, const Layout& L,
                          int* iters_out, hipStream_t s) {
  if (L.rNP == 32)
    return launch_reduced_mfma<T, 32>(n, m, N, k, Xf, Xa, Xg, ng, idx, hw, y, rdiag, eps, tol, maxit, ws,
                                      L, iters_out, s);
  if (L.rNP == 64)
    return launch_reduced_mfma<T, 64>(n, m, N, k, Xf, Xa, Xg, ng, idx, hw, y, rdiag, eps, tol, maxit, ws,
                                      L, iters_out, s);
  if (L.rNP == 128)
    return launch_reduced_mfma<T, 128>(n, m, N, k, Xf, Xa, Xg, ng, idx, hw, y, rdiag, eps, tol, maxit,
                                       ws, L, iters_out, s);
  unsigned char* base = (unsigned char*)ws;
  double* G = (double*)(base + L.rG);
  double* B = (double*)(base + L.rB);
  double* Wd = (double*)(base + L.Wd);
  int* iters = (int*)(base + L.riters);
  int* stat = (int*)(base + L.rstat);
  hipError_t e = red_wide_product<T, false>(ng, m, N, k, Xg, idx, hw, y, rdiag, eps, ws, L, s);
  if (e != hipSuccess) return e;
  if (L.rLG == 192) {
    e = launch_small_cg_x<3, 24>(N, G, B, Wd, iters, iters_out, stat, tol, maxit, s);
  } else if (L.rLG == 256) {  // eight waves of the fewest rows that hold N
    e = N <= 208   ? launch_small_cg_x<4, 26>(N, G, B, Wd, iters, iters_out, stat, tol, maxit, s)
        : N <= 224 ? launch_small_cg_x<4, 28>(N, G, B, Wd, iters, iters_out, stat, tol, maxit, s)
                   : launch_small_cg_x<4, 32>(N, G, B, Wd, iters, iters_out, stat, tol, maxit, s);
  } else {  // N > 256: G no longer fits a CU
    hipLaunchKernelGGL(k_small_cg, dim3(N), dim3(kBlock),
                       sizeof(double) * (4 * (size_t)N + kBlock), s, N, (const double*)G,
                       (const double*)B, Wd, iters, iters_out, stat, tol, maxit);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  return launch_update<T>(n, N, Xf, Xa, Wd, 1, s);
}

// sEnKF analysis (Appendix A, Algorithm 3) with the reduced mode's layout:
// W = Zhat^T diag(Zhat Zhat^T + (N-1) R)^{-1} (Y - Z) from the SEN variants of
// its gather and product kernels and the partial sums (no solve), then
// X_a = X_f + X_f W, Algorithm 3's own form, on the reduced mode's update.
template <typename T, int NP>
hipError_t launch_senkf_mfma(int n, int m, int N, int k, const T* Xf, T* Xa, const int32_t* idx,
                             const T* hw, const T* y, const T* rdiag, const T* eps, void* ws,
                             const Layout& L, int* iters0, hipStream_t s) {
  unsigned char* base = (unsigned char*)ws;
  T* part = (T*)(base + L.rpart);
  int* err = (int*)(base + L.err);
  int* errw = (int*)(base + L.rerr);
  T* Wt = (T*)(base + L.rWt);
  hipError_t e;
  if (red_streamed(m, N, sizeof(T), true)) {
    if ((e = launch_red_stream<T, true>(n, m, N, k, Xf, idx, hw, y, rdiag, eps, ws, L, iters0,
                                        s)) != hipSuccess)
      return e;
  } else if constexpr (NP <= 64) {
    const int S = red_parts(m, N, sizeof(T), true);
    hipLaunchKernelGGL((k_red_pg<T, NP, true>), dim3(S), dim3(kBlock), 0, s, n, m, N, k, Xf,
                       idx, hw, y, rdiag, eps, part, errw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int per = kBlock / 8;
    hipLaunchKernelGGL((k_senkf_sum<T, NP>), dim3((NP * NP + per - 1) / per), dim3(kBlock), 0, s,
                       N, S, (const T*)part, Wt, (const int*)errw, S, err, iters0);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_red_update_np<T, NP>(n, N, Xf, Xa, Wt, s);
}

template <typename T>
hipError_t launch_senkf(int n, int m, int N, int k, const T* Xf, T* Xa, const int32_t* idx,
                        const T* hw, const T* y, const T* rdiag, const T* eps, void* ws,
                        const Layout& L, int* iters0, hipStream_t s) {
  if (L.rNP == 32)
    return launch_senkf_mfma<T, 32>(n, m, N, k, Xf, Xa, idx, hw, y, rdiag, eps, ws, L, iters0, s);
  if (L.rNP == 64)
    return launch_senkf_mfma<T, 64>(n, m, N, k, Xf, Xa, idx, hw, y, rdiag, eps, ws, L, iters0, s);
  if (L.rNP == 128)
    return launch_senkf_mfma<T, 128>(n, m, N, k, Xf, Xa, idx, hw, y, rdiag, eps, ws, L, iters0,
                                     s);
  const hipError_t e = red_wide_product<T, true>(n, m, N, k, Xf, idx, hw, y, rdiag, eps, ws, L, s);
  if (e != hipSuccess) return e;
  if (iters0) {
    const hipError_t ez = launch_zero_u32((unsigned*)iters0, N, s);
    if (ez != hipSuccess) return ez;
  }
  return launch_update<T>(n, N, Xf, Xa, (const double*)((unsigned char*)ws + L.rB), 0, s, nullptr);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_unscale_rows(int m, int N, T* z, const T* rdiag) {
  const long total = (long)m * N;
  for (long e = (long)blockIdx.x * kBlock + threadIdx.x; e < total; e += (long)gridDim.x * kBlock)
    z[e] = (T)((double)z[e] / sqrt((double)rdiag[e / N]));
}

template <typename T>
hipError_t launch_unscale_rows(int m, int N, T* z, const T* rdiag, hipStream_t s) {
  const long total = (long)m * N;
  long nb = (total + kBlock - 1) / kBlock;
  if (nb > 2048) nb = 2048;
  hipLaunchKernelGGL(k_unscale_rows<T>, dim3((unsigned)nb), dim3(kBlock), 0, s, m, N, z, rdiag);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_validate(int n, int m, int N, int k, const T* Xf, const int32_t* idx,
                           const T* hw, const T* y, const T* rdiag, const T* eps, const T* z0,
                           int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_validate<T>, dim3(512), dim3(kBlock), 0, s, n, m, N, k, Xf, idx, hw, y,
                     rdiag, eps, z0, flags);
  return hipGetLastError();
}

#define CGD_INST(T)                                                                              \
  template hipError_t launch_update<T>(int, int, const T*, T*, const double*, int, hipStream_t, \
                                       const int*);                                           \
  template hipError_t launch_reduced<T>(int, int, int, int, const T*, T*, const T*, int,        \
                                        const int32_t*, const T*, const T*, const T*, const T*,  \
                                        double, int, void*, const Layout&, int*, hipStream_t);   \
  template hipError_t launch_validate<T>(int, int, int, int, const T*, const int32_t*, const T*, \
                                         const T*, const T*, const T*, const T*, int*,           \
                                         hipStream_t);                                           \
  template hipError_t launch_unscale_rows<T>(int, int, T*, const T*, hipStream_t);            \
  template hipError_t launch_senkf<T>(int, int, int, int, const T*, T*, const int32_t*, const T*, \
                                      const T*, const T*, const T*, void*, const Layout&, int*,   \
                                      hipStream_t);
CGD_INST(double)
CGD_INST(float)

}  // namespace cgd
