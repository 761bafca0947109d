// Row-block x member-group CG solver in FP64 for 64 < N <= 128 (gfx950):
// the decomposition of cg_tile.hip with members in groups of 16 and 128
// observation rows per workgroup, both S-products on v_mfma_f64_16x16x4f64.
//
// Workgroup (c, b) keeps rows b of S for all members in LDS (130 KiB) and z,
// r, p of group c's 16 members on those rows in registers, as the accumulators
// of Q = S_b G lay them out.  Wave w owns rows 32 w .. of Q and columns 32 w ..
// of the Gram partial S_b^T r, so no partial is summed across waves: r goes to
// the other waves through LDS (in G's place, which the step has used up by
// then).  One exchange per step, summed inside a group as in cg_tile.hip (a
// reduce-scatter and an all-gather through words that carry their exchange
// number); a double is two words, 32 bits of it each, so sums are exact to
// the last bit of the doubles' own addition.  Every workgroup of a group takes
// the same decisions from the same bits; W = sum_k alpha_k G_k in double.
//
// Always launched cooperatively (the workgroups wait for each other); every
// wait is bounded: by 1 s, and in the first exchange, where a workgroup may still be
// waiting for a CU that another stream's kernel holds, by 30 s (the streaming
// solver, which these sizes would run otherwise, waits for that without a bound).
//
// Bound: the exchange (33 KiB out and in per workgroup and step) and 3.4 us of
// FP64 MFMA a step.  16 members a group rather than 32 keep both the
// registers and the exchange of a workgroup at the FP32 solver's size.
// m = 4093, N = 100, k = 2 (90 steps): 24.8 ms on the streaming solver, 4.8 ms
// on the column solver, 1.59 ms here.
#include <atomic>

#include "exchange.h"
#include "internal.h"
#include "mfma_util.h"

namespace cgd {

namespace {

constexpr int kM = 16;            // members per group
constexpr int kRows = 128;        // rows per workgroup
constexpr int kNP = 128;          // padded N
constexpr int kLd = kNP + 2;      // S row stride in LDS (16-byte rows, skewed banks)
constexpr int kGW = kNP * kM;     // doubles of S^T r
constexpr int kEx = kGW + 4 * kM; // doubles of an exchange: S^T r, four sums per member
constexpr int kSlot = 2 * 2 * kEx;  // words per workgroup (two exchanges alternate)
constexpr int kBatch64 = 12;      // owner step: partials in flight per thread
constexpr unsigned long long kFirstWaitTicks = 30 * kTileWaitTicks;

struct __align__(16) T64Lds {
  double S[kRows * kLd];
  double G[kGW];            // G of the step, then r of the step ([row][member])
  double own[kBlock];       // owner step
  double xs[4][kM][4];      // scalar sums per wave
  double gs[4][kM];         // ||G||^2 per wave
  double sums[4 * kM];      // gathered scalar sums
};

struct Tile64Args {
  int N, m, NG, nblk, maxit, want_relres;
  double tol;
  unsigned long long ticks;  // every wait's limit, 0 = kFirstWaitTicks, then kTileWaitTicks
  unsigned long long* txp;  // NG * nblk * kSlot
  unsigned long long* txr;  // NG * kSlot
  const double* S;          // m x kNP
  const double* rv;         // m
  const double* D;          // m x N
  double* z_out;
  int* iters_out;
  double* relres_out;
  double* relres;
  int* coli;
  double* col;
  double* Wd;
  int* err;
};

__device__ inline void st_dbl(unsigned long long* p, double v, unsigned ep) {
  st64(p, (unsigned)__double2loint(v), ep);
  st64(p + 1, (unsigned)__double2hiint(v), ep);
}
__device__ inline double to_dbl(unsigned long long lo, unsigned long long hi) {
  return __hiloint2double((int)(unsigned)hi, (int)(unsigned)lo);
}

__global__ __launch_bounds__(kBlock) void k_cg_tile64(Tile64Args a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T64Lds& L = *reinterpret_cast<T64Lds*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, lr = lane & 15, lk = lane >> 4;
  const int NG = a.NG, nblk = a.nblk, N = a.N, m = a.m;
  const int c = blockIdx.x % NG, b = blockIdx.x / NG, i0 = b * kRows;
  const int j = c * kM + lr;  // this thread's member: lr in the MFMA layouts, tid % 16 in the
  const bool jv = j < N;      // exchange (the same lanes)
  const double inv = 1.0 / (double)(N - 1);
  unsigned long long* mypart = a.txp + (size_t)(c * nblk + b) * kSlot;
  const unsigned long long* gpart = a.txp + (size_t)c * nblk * kSlot;
  unsigned long long* red = a.txr + (size_t)c * kSlot;
  const int dlo = (int)((long)b * kEx / nblk), Ld = (int)((long)(b + 1) * kEx / nblk) - dlo;

  // ---------------- S block; r = d, z = p = 0 ----------------
  for (int e = tid; e < kRows * kNP / 2; e += kBlock) {
    const int i = e / (kNP / 2), c2 = (e - i * (kNP / 2)) * 2, gi = i0 + i;
    v2d x = {0.0, 0.0};
    if (gi < m) x = *reinterpret_cast<const v2d*>(a.S + (size_t)gi * kNP + c2);
    *reinterpret_cast<v2d*>(&L.S[i * kLd + c2]) = x;
  }
  double z[2][4], r[2][4], p[2][4], rv[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int gi = i0 + 32 * wv + 16 * t + frag_row<double>(lk, i);
      r[t][i] = (gi < m && jv) ? a.D[(size_t)gi * N + j] : 0.0;
      rv[t][i] = gi < m ? a.rv[gi] : 0.0;
      z[t][i] = 0.0;
      p[t][i] = 0.0;
    }

  unsigned long long ticks = a.ticks ? a.ticks : kFirstWaitTicks;  // this exchange's limit
  // the four sums of this wave's rows into L.xs
  auto row_sums = [&]() {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double rr = r[t][i], pp = p[t][i], w = rv[t][i];
        v[0] += rr * rr;
        v[1] += w * rr * rr;
        v[2] += w * rr * pp;
        v[3] += w * pp * pp;
      }
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      v[f] += __shfl_xor(v[f], 16);
      v[f] += __shfl_xor(v[f], 32);
      if (lk == 0) L.xs[wv][lr][f] = v[f];
    }
  };
  // Q rows of this wave: S_b G with lane group lk summing columns 8 s + 2 lk + u
  auto product = [&](v4d (&q)[2]) {
    q[0] = v4d{0.0, 0.0, 0.0, 0.0};
    q[1] = q[0];
    const double* s0 = &L.S[(32 * wv + lr) * kLd + 2 * lk];
#pragma unroll 4
    for (int s = 0; s < kNP / 8; ++s) {
      const v2d a0 = *reinterpret_cast<const v2d*>(s0 + 8 * s);
      const v2d a1 = *reinterpret_cast<const v2d*>(s0 + 16 * kLd + 8 * s);
      const double b0 = L.G[(8 * s + 2 * lk) * kM + lr], b1 = L.G[(8 * s + 2 * lk + 1) * kM + lr];
      q[0] = mfma4(a0[0], b0, q[0]);
      q[1] = mfma4(a1[0], b0, q[1]);
      q[0] = mfma4(a0[1], b1, q[0]);
      q[1] = mfma4(a1[1], b1, q[1]);
    }
  };
  // Exchange ep: r to LDS, columns 32 wv .. of S_b^T r, publish with the sums,
  // then this workgroup's slice of all the group's partials.  False when a
  // wait ran out.
  auto exchange = [&](unsigned ep) -> bool {
    __syncthreads();  // every wave is done with G
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        L.G[(32 * wv + 16 * t + frag_row<double>(lk, i)) * kM + lr] = r[t][i];
    row_sums();
    __syncthreads();
    unsigned long long* pp = mypart + (size_t)(ep & 1) * 2 * kEx;
    if (tid < 4 * kM) {
      const int n = tid >> 2, f = tid & 3;
      st_dbl(pp + 2 * (kGW + tid),
             (L.xs[0][n][f] + L.xs[1][n][f]) + (L.xs[2][n][f] + L.xs[3][n][f]), ep);
    }
    v4d g[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    const double* s0 = &L.S[lk * kLd + 32 * wv + lr];
#pragma unroll 8
    for (int s = 0; s < kRows / 4; ++s) {
      const double bv = L.G[(4 * s + lk) * kM + lr];
      g[0] = mfma4(s0[4 * s * kLd], bv, g[0]);
      g[1] = mfma4(s0[4 * s * kLd + 16], bv, g[1]);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st_dbl(pp + 2 * ((32 * wv + 16 * x + frag_row<double>(lk, i)) * kM + lr), g[x][i], ep);
    // owner step: first one word of each partial, then the slice in bulk (see
    // owner_sum in cg_tile.hip)
    const unsigned long long* base = gpart + (size_t)(ep & 1) * 2 * kEx;
    unsigned long long* rp = red + (size_t)(ep & 1) * 2 * kEx;
    bool bad = false;
    for (int q = tid; q < nblk && Ld > 0; q += kBlock) {
      const unsigned long long* w = base + (size_t)q * kSlot + 2 * dlo;
      poll64(w, ep, ld64(w), bad, ticks);
    }
    if (__syncthreads_or(bad)) return false;
    for (int d0 = 0; d0 < Ld; d0 += kBlock) {
      const int nd = min(Ld - d0, kBlock), R = kBlock / nd, sub = tid / nd, x = tid - sub * nd;
      double s = 0.0;
      if (sub < R) {
        const unsigned long long* w0 = base + 2 * (dlo + d0 + x);
        const int q0 = sub * nblk / R, q1 = (sub + 1) * nblk / R;
        for (int q = q0; q < q1; q += kBatch64) {
          unsigned long long w[kBatch64][2];
#pragma unroll
          for (int u = 0; u < kBatch64; ++u)
            if (q + u < q1) {
              w[u][0] = ld64(w0 + (size_t)(q + u) * kSlot);
              w[u][1] = ld64(w0 + (size_t)(q + u) * kSlot + 1);
            }
#pragma unroll
          for (int u = 0; u < kBatch64; ++u)
            if (q + u < q1) {
              const unsigned long long* pw = w0 + (size_t)(q + u) * kSlot;
              const unsigned long long lo = poll64(pw, ep, w[u][0], bad, ticks);
              const unsigned long long hi = poll64(pw + 1, ep, w[u][1], bad, ticks);
              s += to_dbl(lo, hi);
            }
        }
      }
      L.own[tid] = s;
      if (__syncthreads_or(bad)) return false;
      if (tid < nd) {
        double tot = 0.0;
        for (int k = 0; k < R; ++k) tot += L.own[k * nd + tid];
        st_dbl(rp + 2 * (dlo + d0 + tid), tot, ep);
      }
      __syncthreads();
    }
    return true;
  };

  // ---------------- CG ----------------
  const bool need_z = a.z_out != nullptr || a.want_relres;
  const double tol2 = a.tol * a.tol;
  double Gp[8], Wc[8];  // S^T p and W of entries tid + 256 q ([k][member])
#pragma unroll
  for (int q = 0; q < 8; ++q) Gp[q] = Wc[q] = 0.0;
  bool active = jv, fresh = true;
  int iters = 0, status = COL_RUNNING;
  double dn = 0.0, rhoprev = 0.0;
  unsigned ep = 1;
  __syncthreads();  // S is in LDS
  bool bad = !exchange(ep);
  for (int kit = 0; !bad; ++kit) {
    // all-gather: every word once, 16 consecutive bytes per lane
    const unsigned long long* rp = red + (size_t)(ep & 1) * 2 * kEx;
    unsigned long long w[18];
    const int nw = tid < 4 * kM ? 18 : 16;
    auto at = [&](int u) {
      return rp + (u < 16 ? 2 * (tid + kBlock * (u >> 1)) + (u & 1) : 2 * (kGW + tid) + (u & 1));
    };
#pragma unroll
    for (int u = 0; u < 18; ++u)
      if (u < nw) w[u] = ld64(at(u));
    poll_all(w, nw, at, ep, bad, ticks);
    if (tid < 4 * kM) L.sums[tid] = to_dbl(w[16], w[17]);
    if (__syncthreads_or(bad)) {
      bad = true;
      break;
    }
    const double rho = L.sums[4 * lr], ar = L.sums[4 * lr + 1], arp = L.sums[4 * lr + 2],
                 ap = L.sums[4 * lr + 3];
    if (kit == 0) dn = rho;
    int mode = MODE_FROZEN;
    double beta = 0.0;
    if (active) {
      if (rho <= tol2 * dn) {  // ||r|| <= tol ||d||
        active = false;
        status = COL_CONVERGED;
        iters = kit;
      } else if (kit >= a.maxit) {
        active = false;
        status = COL_MAXIT;
        iters = kit;
      } else {
        mode = MODE_STEP;
        beta = fresh ? 0.0 : rho / rhoprev;
      }
    }
    // G = S^T p for p = r + beta p; frozen members take 0
    double gg = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double x = to_dbl(w[2 * q], w[2 * q + 1]);
      const double gd = mode == MODE_STEP ? (beta != 0.0 ? fma(beta, Gp[q], x) : x) : 0.0;
      Gp[q] = gd;
      gg += gd * gd;
      L.G[tid + kBlock * q] = gd;
    }
    gg += __shfl_xor(gg, 16);
    gg += __shfl_xor(gg, 32);
    if (lk == 0) L.gs[wv][lr] = gg;
    if (!__syncthreads_or(mode == MODE_STEP)) break;  // every member of the group is done
    gg = (L.gs[0][lr] + L.gs[1][lr]) + (L.gs[2][lr] + L.gs[3][lr]);
    double alpha = 0.0;
    if (mode == MODE_STEP) {
      alpha = rho / (gg * inv + ar + 2.0 * beta * arp + beta * beta * ap);
      rhoprev = rho;
      fresh = false;
      if (!isfinite(alpha) || !isfinite(beta)) {
        active = false;
        status = COL_NONFINITE;
        iters = kit;
        mode = MODE_FROZEN;
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) Wc[q] += alpha * Gp[q];
      }
    }
    v4d qa[2];
    product(qa);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (mode == MODE_STEP) {
          const double pn = beta != 0.0 ? fma(beta, p[t][i], r[t][i]) : r[t][i];
          const double q = qa[t][i] * inv + rv[t][i] * pn;
          p[t][i] = pn;
          if (need_z) z[t][i] += alpha * pn;
          r[t][i] -= alpha * q;
        }
    ++ep;
    if (kit == 0) ticks = a.ticks ? a.ticks : kTileWaitTicks;
    bad = !exchange(ep);
  }
  if (bad) {
    if (tid == 0) atomicOr(a.err, 1);
    return;
  }

  // ---------------- results ----------------
  if (b == 0) {
    if (tid < kM && jv) {
      a.coli[CI_ITERS * N + j] = iters;
      a.coli[CI_STATUS * N + j] = status;
      a.coli[CI_FALLBACK * N + j] = 0;
      a.col[CF_DN * N + j] = dn;
      if (a.iters_out) a.iters_out[j] = iters;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = (tid + kBlock * q) / kM;
      if (k < N && jv) a.Wd[(size_t)k * N + j] = Wc[q] * inv;
    }
  }
  if (a.z_out && jv)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int gi = i0 + 32 * wv + 16 * t + frag_row<double>(lk, i);
        if (gi < m) a.z_out[(size_t)gi * N + j] = z[t][i];
      }
  if (!a.want_relres) return;
  // true residual d - S W - R z, its squared norm summed by workgroup b = 0
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 8; ++q) L.G[tid + kBlock * q] = Wc[q] * inv;
  __syncthreads();
  v4d qa[2];
  product(qa);
  double v = 0.0;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int gi = i0 + 32 * wv + 16 * t + frag_row<double>(lk, i);
      if (gi < m && jv) {
        const double res = a.D[(size_t)gi * N + j] - qa[t][i] - rv[t][i] * z[t][i];
        v += res * res;
      }
    }
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  if (lk == 0) L.gs[wv][lr] = v;
  __syncthreads();
  const unsigned er = ep + 1;
  if (tid < kM)
    st_dbl(mypart + (size_t)(er & 1) * 2 * kEx + 2 * tid,
           (L.gs[0][lr] + L.gs[1][lr]) + (L.gs[2][lr] + L.gs[3][lr]), er);
  if (b != 0) return;
  double tot = 0.0;
  for (int q = tid / kM; q < nblk; q += kBlock / kM) {
    const unsigned long long* w = gpart + (size_t)q * kSlot + (size_t)(er & 1) * 2 * kEx + 2 * lr;
    const unsigned long long lo = poll64(w, er, ld64(w), bad, ticks);
    const unsigned long long hi = poll64(w + 1, er, ld64(w + 1), bad, ticks);
    tot += to_dbl(lo, hi);
  }
  L.own[tid] = tot;
  if (__syncthreads_or(bad)) {
    if (tid == 0) atomicOr(a.err, 1);
    return;
  }
  if (tid < kM && jv) {
    tot = 0.0;
    for (int k = 0; k < kBlock / kM; ++k) tot += L.own[k * kM + tid];
    const double rr2 = dn > 0 ? sqrt(tot / dn) : 0.0;
    a.relres[j] = rr2;
    if (a.relres_out) a.relres_out[j] = rr2;
  }
}

// S (m x kNP, zero past N), D (m x N) and the rows' diag(R), one wave per row
// (two members per lane); scaled rows and unit R when preconditioned.
__global__ __launch_bounds__(kBlock) void k_tile64_gather(CGArgs<double> a, double* S, double* D,
                                                          double* rv) {
  const int lane = threadIdx.x & 63, gi = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int N = a.N;
  if (gi >= a.m) return;
  double h[2] = {0.0, 0.0};
  for (int t = 0; t < a.k; ++t) {
    const int src = a.idx[(size_t)gi * a.k + t];
    const double wt = a.hw[(size_t)gi * a.k + t];
    if ((unsigned)src >= (unsigned)a.ng) {
      if (lane == 0) atomicOr(a.err, 2);
      continue;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (lane + 64 * u < N) h[u] += wt * a.Xg[(size_t)src * N + lane + 64 * u];
  }
  const double mean = wave_sum(h[0] + h[1]) / (double)N;
  const double sc = precond_row_scale(a, gi), yv = a.y[gi];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int col = lane + 64 * u;
    const bool on = col < N;
    S[(size_t)gi * kNP + col] = on ? (h[u] - mean) * sc : 0.0;
    if (on) {
      double d = yv - h[u];
      if (a.eps) d += a.eps[(size_t)gi * N + col];
      D[(size_t)gi * N + col] = d * sc;
    }
  }
  if (lane == 0) rv[gi] = effective_r(a, gi);
}

}  // namespace

int tile64_shape(int m, int N, int* NG, int* nblk) {
  if (N <= 64 || N > kNP || m < 1) return 0;
  *NG = (N + kM - 1) / kM;
  *nblk = (m + kRows - 1) / kRows;
  return 1;
}

size_t tile64_words(int NG, int nblk) { return (size_t)kSlot * NG * (nblk + 1); }

// Workgroups that run at once on the current device (asked once per device;
// 0 where it cannot be had).
int tile64_coresident() {
  constexpr int kDevs = 64;
  static std::atomic<int> known[kDevs];  // value + 1
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return 0;
  const int k = known[dev].load(std::memory_order_relaxed);
  if (k > 0) return k - 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipFuncSetAttribute((const void*)k_cg_tile64, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)sizeof(T64Lds)) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_cg_tile64, kBlock, sizeof(T64Lds)) !=
          hipSuccess)
    return 0;
  known[dev].store(per * cus + 1, std::memory_order_relaxed);
  return per * cus;
}

hipError_t launch_cg_tile64(const CGArgs<double>& a, int NG, int nblk, unsigned long long* words,
                            double* S, double* D, double* rv, hipEvent_t* ev, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_words, dim3(1024), dim3(kBlock), 0, s, words,
                     tile64_words(NG, nblk));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_zero_u32((unsigned*)a.err, 1, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_tile64_gather, dim3((a.m + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock),
                     0, s, a, S, D, rv);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;  // the solver launch alone
  if ((e = hipFuncSetAttribute((const void*)k_cg_tile64,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(T64Lds))) != hipSuccess)
    return e;
  Tile64Args t;
  t.N = a.N;
  t.m = a.m;
  t.NG = NG;
  t.nblk = nblk;
  t.maxit = a.maxit;
  t.want_relres = a.want_relres;
  t.tol = a.tol;
  t.ticks = a.census_ticks;
  t.txp = words;
  t.txr = words + (size_t)kSlot * NG * nblk;
  t.S = S;
  t.rv = rv;
  t.D = D;
  t.z_out = a.z_out;
  t.iters_out = a.iters_out;
  t.relres_out = a.relres_out;
  t.relres = a.relres;
  t.coli = a.coli;
  t.col = a.col;
  t.Wd = a.Wd;
  t.err = a.err;
  void* args[] = {&t};
  return hipLaunchCooperativeKernel((const void*)k_cg_tile64, dim3(NG * nblk), dim3(kBlock), args,
                                    (unsigned)sizeof(T64Lds), s);
}

}  // namespace cgd
