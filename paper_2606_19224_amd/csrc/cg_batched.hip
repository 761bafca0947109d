// Batched mode in FP32 (gfx950), batches that fill the GPU: the CG of four members
// of a filter per workgroup, with both S-products on v_mfma_f32_4x4x1_16b_f32.
//
// That MFMA forms sixteen 4 x 4 outer products at the rate of the larger FP32
// shapes, and can broadcast one block's A operand to all sixteen.  With the
// four members as the A rows, a wave takes 64 observation rows at a time:
//
//  * q = S g, one MFMA per column k of S: lane = row supplies S[row][k], the
//    broadcast block supplies g[k] of the four members.  A lane ends with q of
//    its own row for the four members, which is how r and p lie in memory
//    ([group of four members][row][4]: one 16-byte access per lane);
//  * S^T r, one MFMA per row (per two or four rows when 32 or 16 columns
//    leave blocks free): lane = column supplies S[row][k], the broadcast block
//    r[row] of the four members, which a 4 x 4 transpose inside each quad of
//    lanes puts in place.  A lane ends with the four members' sums of its
//    column.
//
// S comes from memory once per pass, as [k / 4][row][4] (a lane's 16 bytes, 1
// KiB per wave load), and goes through the wave's own LDS tile for the second
// product.  The next tile's loads are in flight during the second product.
// The products' chains of FP32 sums stay within one tile (at most 16 terms each
// way of the four accumulators); their tiles and waves are added in double, in a
// fixed order.  The scalar sums (r.r, r.Rr, r.Rp, p.Rp) add a lane's rows in FP32, one
// a tile of its wave (m / 512 terms; the per-member solver as many or twice that),
// then lanes and waves in double.  No workgroup waits for another.
//
// Bound: the MFMA, LDS and L2 paths of a tile are within a factor of two of
// each other.  One workgroup per member on the vector ALUs re-read S from L2
// for every member and was bound by that: 64 filters of 1024 to 32768
// variables took 961 us in the solve; four members per workgroup take 615 us
// (and 111 -> 67 us for the gather, which no longer writes a second layout).
// 12 waves with half tiles each spilled (942 us).  The sums by halving exchanges
// and the first tile's S requested before the decisions matter where a wave has
// one tile: 8 filters of up to 2048 variables, whole call 131 us without and 106
// us with both (124 us one workgroup per member).
#include <type_traits>
#include <utility>

#include "internal.h"
#include "mfma_util.h"

namespace cgd {

namespace {

constexpr int kBT = 512;           // threads per workgroup
constexpr int kBW = kBT / 64;      // waves
constexpr int kTR = 64;            // rows per tile

template <int NP>
struct BM {
  static constexpr int NQ = NP / 4;       // 16-byte chunks of a row
  static constexpr int G = 64 / NP;       // rows per MFMA of the second product
  static constexpr int CB = NP == 64 ? 4 : NP == 32 ? 3 : 2;  // its broadcast size
  static constexpr int LDT = NP + 4;      // row stride of a wave's LDS tile
};

struct BShared {
  double wsum[kBW][16];   // per wave: four sums of four members
  double gpart[4][4];     // ||G||^2 per deciding wave and member
  float g4[64 * 4];       // G of the step, [k][member]
  float al[4], be[4];
  int mode[4];
};
constexpr size_t kBTile = sizeof(float) * kTR * (64 + 4);  // a wave's tile at NP = 64
constexpr size_t kBLds = kBW * kBTile;                     // (its head holds the wave's sums after a pass)
static_assert(kBTile >= sizeof(double) * 64 * 4, "a wave's sums fit its tile");

template <int CB, int AB>
__device__ inline v4f mfma_b(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CB, AB, 0);
}
template <typename F, int... I>
__device__ __attribute__((always_inline)) inline void each(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// Lane i of the quad, to all four lanes of it.
template <int I>
__device__ inline float quad(float v) {
  return dpp<I * 0x55>(v);
}

// Sum of v[lane % 16] over the wave, in double, from every lane's 16 values: each
// exchange halves the values a lane keeps (15 exchanges and two more across the
// rows of 16 lanes, where a tree per value takes six each).
__device__ __attribute__((always_inline)) inline double wave_sums16(const double (&v)[16],
                                                                    int lane) {
  double a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool hi = lane & 8;
    a[i] = (hi ? v[8 + i] : v[i]) + dpp<0x140>(hi ? v[i] : v[8 + i]);  // row_mirror
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool hi = lane & 4;
    b[i] = (hi ? a[4 + i] : a[i]) + dpp<0x141>(hi ? a[i] : a[4 + i]);  // row_half_mirror
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool hi = lane & 2;
    c[i] = (hi ? b[2 + i] : b[i]) + dpp<0x4E>(hi ? b[i] : b[2 + i]);   // lane ^ 2
  }
  const bool hi = lane & 1;
  double d = (hi ? c[1] : c[0]) + dpp<0xB1>(hi ? c[0] : c[1]);         // lane ^ 1
  d += __shfl_xor(d, 16);
  return d + __shfl_xor(d, 32);
}

// A wave's rows of a tile.  S of its first tile is requested at the end of the
// pass before, so that the decisions between two passes cover the latency (r
// and p as well would spill).
template <int NP>
struct BmTile {
  v4f s[BM<NP>::NQ], r, p;
  float w;
};
template <int NP>
__device__ __attribute__((always_inline)) inline void bm_load_s(int mp, const float* S, int t,
                                                                BmTile<NP>& x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < BM<NP>::NQ; ++q)
    x.s[q] = *reinterpret_cast<const v4f*>(S + ((size_t)q * mp + t * kTR + lane) * 4);
}
template <int NP>
__device__ __attribute__((always_inline)) inline void bm_load_v(bool step, const float* R4,
                                                                const float* P4, const float* rv,
                                                                int t, BmTile<NP>& x) {
  const int i = t * kTR + (threadIdx.x & 63);
  x.r = *reinterpret_cast<const v4f*>(R4 + (size_t)i * 4);
  if (step) x.p = *reinterpret_cast<const v4f*>(P4 + (size_t)i * 4);
  x.w = rv[i];
}

// One pass over the problem's rows, S of the first tile in x.  STEP: p = r + beta p, q = S g/(N-1) + R
// p, r -= alpha q first (gr: this lane's g, entry e of lane 4 q + m is g[4 q
// + e] of member m); else r = d as it lies in memory.  Leaves this wave's part
// of S^T r in its tile ([lane][member], lane % NP the column) and its sums
// (r.r, r.Rr, r.Rp, p.Rp per member) in sh.wsum.
template <int NP, bool STEP>
__device__ __attribute__((always_inline)) inline void bm_pass(
    int mp, const float* S, float* R4, float* P4, const float* rv, float inv, const float (&gr)[4],
    BShared& sh, float* tile, BmTile<NP>& x) {
  using C = BM<NP>;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nt = mp / kTR;
  const int n = lane & 3;
  float al[4], be[4];
  bool on[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    al[m] = STEP ? sh.al[m] : 0.f;
    be[m] = STEP ? sh.be[m] : 0.f;
    on[m] = STEP && sh.mode[m] == MODE_STEP;
  }
  double gd[4] = {0.0, 0.0, 0.0, 0.0};
  float sm[4][4];  // (one row per tile and lane; lanes and waves in double)
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int f = 0; f < 4; ++f) sm[m][f] = 0.f;
  int t = wv;
  if (t < nt) bm_load_v<NP>(STEP, R4, P4, rv, t, x);
  for (; t < nt; t += kBW) {
    // S rows to the LDS tile, and the first product from the registers
#pragma unroll
    for (int q = 0; q < C::NQ; ++q) *reinterpret_cast<v4f*>(tile + lane * C::LDT + 4 * q) = x.s[q];
    v4f qa[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) qa[e] = v4f{0, 0, 0, 0};
    if constexpr (STEP)
      each(std::make_integer_sequence<int, C::NQ>{}, [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int e = 0; e < 4; ++e) qa[e] = mfma_b<4, q>(gr[e], x.s[q][e], qa[e]);
      });
    if (t + kBW < nt) bm_load_s<NP>(mp, S, t + kBW, x);
    v4f rn = x.r, pn = v4f{0, 0, 0, 0};
    const float wr = x.w;
    if constexpr (STEP) {
      const v4f qs = (qa[0] + qa[1]) + (qa[2] + qa[3]);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        pn[m] = be[m] != 0.f ? x.r[m] + be[m] * x.p[m] : x.r[m];  // (p is not set before the first step)
        const float q = qs[m] * inv + wr * pn[m];
        rn[m] = on[m] ? x.r[m] - al[m] * q : x.r[m];
      }
      *reinterpret_cast<v4f*>(R4 + (size_t)(t * kTR + lane) * 4) = rn;
      *reinterpret_cast<v4f*>(P4 + (size_t)(t * kTR + lane) * 4) = pn;
    }
    if (t + kBW < nt) bm_load_v<NP>(STEP, R4, P4, rv, t + kBW, x);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float rr = wr * rn[m];
      sm[m][0] += rn[m] * rn[m];
      sm[m][1] += rr * rn[m];
      if constexpr (STEP) {
        sm[m][2] += rr * pn[m];
        sm[m][3] += wr * pn[m] * pn[m];
      }
    }
    // ra[i] in lane 4 b + m: r of row 4 b + i, member m
    float ra[4];
    each(std::make_integer_sequence<int, 4>{}, [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      const float x0 = quad<i>(rn[0]), x1 = quad<i>(rn[1]), x2 = quad<i>(rn[2]),
                  x3 = quad<i>(rn[3]);
      const float a = (n & 1) ? x1 : x0, b = (n & 1) ? x3 : x2;
      ra[i] = (n & 2) ? b : a;
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // rows 4 b + i (+ 64 / G per further group of lanes)
    v4f ga[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ga[i] = v4f{0, 0, 0, 0};
    const float* col = tile + (lane / NP) * NP * C::LDT + lane % NP;
    each(std::make_integer_sequence<int, NP / 4>{}, [&](auto bc) __attribute__((always_inline)) {
      constexpr int b = decltype(bc)::value;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        ga[i] = mfma_b<C::CB, b>(ra[i], col[(4 * b + i) * C::LDT], ga[i]);
    });
    const v4f g = (ga[0] + ga[1]) + (ga[2] + ga[3]);
#pragma unroll
    for (int m = 0; m < 4; ++m) gd[m] += (double)g[m];
    // (the next tile's stores come after this tile's reads: LDS is in order)
    __builtin_amdgcn_wave_barrier();
  }
  double* red = reinterpret_cast<double*>(tile);
#pragma unroll
  for (int m = 0; m < 4; ++m) red[lane * 4 + m] = gd[m];
  double v[16];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int f = 0; f < 4; ++f) v[4 * m + f] = (double)sm[m][f];
  const double sum = wave_sums16(v, lane);
  if (lane < 16) sh.wsum[wv][lane] = sum;
  __builtin_amdgcn_sched_barrier(0);  // (earlier, the tile's registers would spill)
  if (wv < nt) {
    bm_load_s<NP>(mp, S, wv, x);
  }
}

// Four members 4 g .. of one problem.
template <int NP>
__device__ __attribute__((always_inline)) inline void bm_solve(const BProb<float>& P, int g,
                                                               double tol, int maxit,
                                                               unsigned char* smem, BShared& sh) {
  using C = BM<NP>;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, N = P.N;
  float* tile = (float*)(smem + wv * kBTile);
  float* R4 = P.Vr + (size_t)g * P.mp * 4;
  float* P4 = P.Vp + (size_t)g * P.mp * 4;
  const double inv = 1.0 / (double)(N - 1);
  const bool dec = tid < NP * 4;  // deciding threads: column k = tid / 4, member m = tid % 4
  const int m = tid & 3, k = tid >> 2, j = 4 * g + m;
  double Gc = 0.0, Wc = 0.0, dn = 0.0, rhoprev = 0.0;
  bool active = true, fresh = true;
  int iters = 0, status = COL_RUNNING;
  float gr[4] = {0.f, 0.f, 0.f, 0.f};
  BmTile<NP> x;
  if (wv < P.mp / kTR) bm_load_s<NP>(P.mp, P.Sp, wv, x);
  bm_pass<NP, false>(P.mp, P.Sp, R4, P4, P.Rp, (float)inv, gr, sh, tile, x);
  for (int kit = 0;; ++kit) {
    __syncthreads();
    double rho = 0.0, sa = 0.0, sb = 0.0, sc = 0.0, gk = 0.0, beta = 0.0;
    int mode = MODE_FROZEN;
    if (dec) {
      double Gr = 0.0;
#pragma unroll
      for (int w = 0; w < kBW; ++w) {
        const double* red = reinterpret_cast<const double*>(smem + w * kBTile);
#pragma unroll
        for (int h = 0; h < C::G; ++h) Gr += red[(k + h * NP) * 4 + m];
        rho += sh.wsum[w][4 * m];
        sa += sh.wsum[w][4 * m + 1];
        sb += sh.wsum[w][4 * m + 2];
        sc += sh.wsum[w][4 * m + 3];
      }
      if (kit == 0) dn = rho;
      if (active) {
        if (sqrt(rho) <= tol * sqrt(dn)) {
          active = false;
          status = COL_CONVERGED;
          iters = kit;
        } else if (kit >= maxit) {
          active = false;
          status = COL_MAXIT;
          iters = kit;
        } else {
          mode = MODE_STEP;
          beta = fresh ? 0.0 : rho / rhoprev;
        }
      }
      // G = S^T p as the products use it, and its squared norm
      if (mode == MODE_STEP) gk = (double)(float)(beta != 0.0 ? Gr + beta * Gc : Gr);
      sh.g4[tid] = (float)gk;
      double gsq = gk * gk;
      gsq += __shfl_xor(gsq, 4);
      gsq += __shfl_xor(gsq, 8);
      gsq += __shfl_xor(gsq, 16);
      gsq += __shfl_xor(gsq, 32);
      if (lane < 4) sh.gpart[wv][lane] = gsq;
    }
    __syncthreads();
    if (dec) {
      double gg = 0.0, alpha = 0.0;
      for (int w = 0; w < NP / 16; ++w) gg += sh.gpart[w][m];
      if (mode == MODE_STEP) {
        alpha = rho / (gg * inv + sa + 2.0 * beta * sb + beta * beta * sc);
        if (!isfinite(alpha) || !isfinite(beta)) {
          active = false;
          status = COL_NONFINITE;
          iters = kit;
          mode = MODE_FROZEN;
          alpha = 0.0;
        } else {
          Gc = gk;
          Wc += alpha * gk;
          rhoprev = rho;
          fresh = false;
        }
      }
      if (k == 0) {
        sh.al[m] = (float)alpha;
        sh.be[m] = (float)beta;
        sh.mode[m] = mode;
      }
    }
    __syncthreads();
    if (sh.mode[0] != MODE_STEP && sh.mode[1] != MODE_STEP && sh.mode[2] != MODE_STEP &&
        sh.mode[3] != MODE_STEP)
      break;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      gr[e] = lane < NP ? sh.g4[((lane & ~3) + e) * 4 + (lane & 3)] : 0.f;
    bm_pass<NP, true>(P.mp, P.Sp, R4, P4, P.Rp, (float)inv, gr, sh, tile, x);
  }
  if (!dec || j >= N) return;
  if (k < N) P.Wd[(size_t)k * N + j] = Wc * inv;
  if (k == 0) {
    P.coli[CI_ITERS * N + j] = iters;
    P.coli[CI_STATUS * N + j] = status;
    P.coli[CI_FALLBACK * N + j] = 0;
    P.col[CF_DN * N + j] = dn;
    if (P.iters_out) P.iters_out[j] = iters;
  }
}

__global__ __launch_bounds__(kBT) void k_bm_solve(const BProb<float>* probs, const int2* tab,
                                                  double tol, int maxit) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ BShared sh;
  const int2 ent = tab[blockIdx.x];
  if (ent.x < 0) return;  // padding of an XCD queue
  const BProb<float> P = probs[ent.x];
  switch (P.NP) {
    case 16: bm_solve<16>(P, ent.y, tol, maxit, smem_raw, sh); break;
    case 32: bm_solve<32>(P, ent.y, tol, maxit, smem_raw, sh); break;
    default: bm_solve<64>(P, ent.y, tol, maxit, smem_raw, sh); break;
  }
}

// Rows [ent.y, ent.y + gr) of a problem: HX (double), S and D = r, both as
// [chunk of four members][row][4], and diag(R) (0 past m).  NP/4 lanes per row;
// two row steps' loads in flight.
template <int NP>
__device__ __attribute__((always_inline)) inline void bm_gather(const BProb<float>& P, int ib, int ie,
                                                                int precond, int* err) {
  constexpr int LPR = NP / 4, RPS = kBT / LPR, U = 2;
  const int tid = threadIdx.x, q = tid % LPR, rw = tid / LPR, c0 = 4 * q;
  const int N = P.N, m = P.m, mp = P.mp;
  for (int s0 = ib; s0 < ie; s0 += U * RPS) {
    double h[U][4], yv[U], rv[U];
    float ev[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = s0 + u * RPS + rw;
      const bool live = i < ie && i < m;
      yv[u] = live ? (double)P.y[i] : 0.0;
      rv[u] = live ? (double)P.rdiag[i] : 1.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        h[u][c] = 0.0;
        ev[u][c] = (live && P.eps && c0 + c < N) ? P.eps[(size_t)i * N + c0 + c] : 0.f;
      }
    }
    for (int t = 0; t < P.k; ++t) {
      int col[U];
      double wt[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = s0 + u * RPS + rw;
        col[u] = 0;
        wt[u] = 0.0;
        if (i < ie && i < m) {
          const int cx = P.idx[(size_t)i * P.k + t];
          if ((unsigned)cx < (unsigned)P.n) {
            col[u] = cx;
            wt[u] = (double)P.hw[(size_t)i * P.k + t];
          } else {
            atomicOr(err, 2);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c0 + c < N) h[u][c] += wt[u] * (double)P.Xf[(size_t)col[u] * N + c0 + c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = s0 + u * RPS + rw;
      const double mean = group_sum<LPR>((h[u][0] + h[u][1]) + (h[u][2] + h[u][3])) / N;
      if (i < ie) {
        const double sc = precond ? 1.0 / sqrt(rv[u]) : 1.0;
        v4f s, d;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bool live = i < m && c0 + c < N;
          s[c] = live ? (float)((h[u][c] - mean) * sc) : 0.f;
          d[c] = live ? (float)((yv[u] - h[u][c] + (double)ev[u][c]) * sc) : 0.f;
        }
        *reinterpret_cast<v4f*>(P.Sp + ((size_t)q * mp + i) * 4) = s;
        if (c0 < N) *reinterpret_cast<v4f*>(P.Vr + ((size_t)q * mp + i) * 4) = d;
        if (q == 0) P.Rp[i] = i < m ? (precond ? 1.f : (float)rv[u]) : 0.f;
      }
    }
  }
}

__global__ __launch_bounds__(kBT) void k_bm_gather(const BProb<float>* probs, const int2* tab,
                                                   int* err, int precond) {
  const int2 ent = tab[blockIdx.x];
  const BProb<float> P = probs[ent.x];
  const int ie = min(P.mp, ent.y + P.gr);
  switch (P.NP) {
    case 16: bm_gather<16>(P, ent.y, ie, precond, err); break;
    case 32: bm_gather<32>(P, ent.y, ie, precond, err); break;
    default: bm_gather<64>(P, ent.y, ie, precond, err); break;
  }
}

}  // namespace

int batched_groups(int N) { return (N + 3) / 4; }

int batched_rows(int m) {
  return m > kColumnsMaxRows ? 0 : (m + kTR - 1) / kTR * kTR;
}

hipError_t launch_bm(const BProb<float>* probs, const int2* gtab, int ngather, const int2* stab,
                     int nsolve, double tol, int maxit, int precond, int* err, hipEvent_t* ev,
                     hipStream_t s) {
  hipError_t e;
  hipLaunchKernelGGL(k_bm_gather, dim3(ngather), dim3(kBT), 0, s, probs, gtab, err, precond);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // profiling events bracket the CG launch alone
  if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
  if ((e = hipFuncSetAttribute((const void*)k_bm_solve,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBLds)) !=
      hipSuccess)
    return e;
  hipLaunchKernelGGL(k_bm_solve, dim3(nsolve), dim3(kBT), kBLds, s, probs, stab, tol, maxit);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return ev ? hipEventRecord(ev[1], s) : hipSuccess;
}

}  // namespace cgd
