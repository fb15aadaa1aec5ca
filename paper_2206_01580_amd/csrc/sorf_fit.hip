// Fit of one element's projection (arXiv 2206.01580, Theory section, SORF
// subsection: Z~_e = U_e S_e V_e^T over sampled representations, U_e^{N_PCA}
// its first N_PCA columns). The left singular vectors of Z~_e are the
// eigenvectors of G = Z~_e Z~_e^T = sum over the sampled rows of rho^T rho
// (n x n, n = d_rep), and the singular values the square roots of its
// eigenvalues. G is formed in FP64 by the FP64 Gram kernel; only its n_pca
// largest eigenpairs are computed, all in FP64:
//
//   tridiagonal  Householder reduction Q^T G Q = T, one launch per column. A
//                launch applies the previous column's rank-two update to its
//                rows and multiplies the updated rows by the new reflector in
//                the same pass, so a column costs one read and one write of
//                the trailing matrix (L2-resident) and one launch;
//   bisect       one workgroup per wanted eigenvalue of T: every thread counts
//                the eigenvalues below its own shift (Sturm sequence), so a pass
//                narrows the interval 257-fold and seven or eight passes reach
//                the rounding of T;
//   vectors      inverse iteration on T (LU with partial pivoting), one wave
//                per vector;
//   clusters     vectors of eigenvalues closer than kFitCluster ||T|| are
//                orthonormalised in order, one workgroup per 16; their inverse
//                iteration is repeated from the orthonormal vectors. Nothing to
//                do where the wanted spectrum decays slowly; for n_pca above the
//                rank of the sample it is most of the call (44 ms at n = n_pca =
//                720 and rank 100);
//   back         the reflectors are applied to the wanted vectors only.
//
// What bounds it: the chain of n dependent columns, each a launch of about six
// microseconds (launch, two workgroup sums, one pass over L2; the arithmetic is
// under 2 % of that). At n = 720, n_pca = 128 (1000 samples) the call takes
// 5.4 ms: columns 4.2, vectors 0.54, back 0.46, bisection 0.29, Gram 0.05. The
// cyclic Jacobi method that stood here before took 112 ms (15 sweeps of 719
// launches, all n eigenvectors rotated at every one of them; with blocks of 16
// indices it needs as many sweeps, so fewer launches alone would not do).
#include "sorf_internal.h"

namespace sorf {

constexpr int kFitThreads = 256;
constexpr int kFitLdsN = 1600;           // largest n whose LU factors stay in LDS (40 n bytes)
constexpr int kFitPasses = 10;           // 257^8 = 2^64: the interval is at rounding size by then
constexpr double kFitEps = 2.220446049250313e-16;
// Vectors of eigenvalues further apart than this (relative to ||T||) are
// orthogonal to eps / kFitCluster = 2e-8 by themselves, below the rounding of
// the FP32 output.
constexpr double kFitCluster = 1e-8;
// Squared length below which a column counts as reduced already. G's entries are
// sums of products of FP32 numbers, so a G that is not zero has a norm of 1e-90
// or more and 1e-140 is far below its rounding; the squares above it are far
// from the end of the FP64 range.
constexpr double kFitNothing = 1e-280;

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over a wave, the same value in every lane: butterflies inside each row
// of 16 lanes (no LDS round trip: this is on the chain of every column and
// every reflector), then the four row sums.
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0xB1>(v);    // lane ^ 1
  v = dpp_add<0x4E>(v);    // lane ^ 2
  v = dpp_add<0x141>(v);   // mirrored half rows: the other quad
  v = dpp_add<0x140>(v);   // mirrored rows: the other half
  auto row = [&](int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
  };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// Sum over the workgroup's four waves, the same value in every thread.
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return v;
}

// 1 / q to rounding (the hardware's approximation, two Newton steps).
__device__ __forceinline__ double fit_rcp(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(r, fma(-q, r, 1.0), r);
  return fma(r, fma(-q, r, 1.0), r);
}

// A (n x n, full) = the symmetric matrix whose lower triangle is G.
__global__ __launch_bounds__(256) void fit_init_kernel(const double* __restrict__ G, int n,
                                                       double* __restrict__ A) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= int64_t(n) * n) return;
  const int i = int(t / n), j = int(t % n);
  A[t] = i >= j ? G[t] : G[int64_t(j) * n + i];
}

// Column k of the reduction. In: A with the updates of columns < k - 1, the
// reflector v of column k - 1 (H = I - tau v v^T, entries >= k, the first one 1,
// so that 1 <= tau <= 2 however small the column was), tau and p = A v. Every
// workgroup forms, from row k of A and these vectors,
//   w = tau p - (tau^2 / 2) (v . p) v,   column k of A - v w^T - w v^T,
// the diagonal entry, the subdiagonal entry and the next reflector; then it
// updates its own rows i > k and multiplies them by the new reflector. Row k
// itself is read by all and written by none.
template <int NMAX>
__global__ __launch_bounds__(kFitThreads) void fit_column_kernel(
    double* __restrict__ A, int n, int k, const double* __restrict__ p_in,
    double* __restrict__ p_out, double* __restrict__ Vh, double* __restrict__ tau,
    double* __restrict__ diag, double* __restrict__ sub) {
  __shared__ double sv[NMAX], sw[NMAX], sn[NMAX];   // old reflector, w, new reflector
  __shared__ double red[4];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int i = k + 1 + ((int(blockIdx.x) * kFitThreads + tid) >> 6);   // this wave's row
  double* __restrict__ Ai = A + int64_t(i < n ? i : n - 1) * n;
  // the row is requested first, to arrive while the reflector is formed
  constexpr int EPT = NMAX / 64;
  constexpr bool HELD = EPT <= 16;
  double ai[HELD ? EPT : 1];
  if constexpr (HELD) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int j = e * 64 + lane;
      ai[e] = j > k && j < n ? Ai[j] : 0.0;
    }
  }
  const double tau0 = k > 0 ? tau[k - 1] : 0.0;
  const double* __restrict__ row = A + int64_t(k) * n;
  const double* __restrict__ v0 = Vh + int64_t(k > 0 ? k - 1 : 0) * n;
  double vp = 0.0;
  for (int j = k + tid; j < n; j += kFitThreads) {
    const double v = k > 0 ? v0[j] : 0.0;
    const double p = k > 0 ? p_in[j] : 0.0;
    sv[j] = v;
    sw[j] = p;
    vp = fma(v, p, vp);
  }
  vp = block_sum(vp, red);
  const double half = 0.5 * tau0 * tau0 * vp;
  for (int j = k + tid; j < n; j += kFitThreads) sw[j] = tau0 * sw[j] - half * sv[j];
  __syncthreads();
  const double vk = sv[k], wk = sw[k];
  double x2 = 0.0;   // squared norm of the column below the subdiagonal entry
  for (int j = k + tid; j < n; j += kFitThreads) {
    const double c = row[j] - (sv[j] * wk + sw[j] * vk);
    sn[j] = c;
    if (j > k + 1) x2 = fma(c, c, x2);
  }
  x2 = block_sum(x2, red);
  const double dk = sn[k];
  const double x0 = k + 1 < n ? sn[k + 1] : 0.0;
  // sn: the reflector times its head; the scale is put into what leaves the kernel
  double t = 0.0, alpha = x0, scale = 1.0;
  if (x2 > kFitNothing) {
    const double norm = sqrt(fma(x0, x0, x2));
    alpha = x0 > 0.0 ? -norm : norm;
    const double head = x0 - alpha, h2 = head * head;   // |head| >= norm
    t = 2.0 * h2 * fit_rcp(h2 + x2);
    scale = fit_rcp(head);
    __syncthreads();                            // x0 has been read by every thread
    if (tid == 0) sn[k + 1] = head;
  } else if (x2 != x2) {
    t = x2;                                     // not a number: carried into the result
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int j = k + 1 + tid; j < n; j += kFitThreads) Vh[int64_t(k) * n + j] = sn[j] * scale;
    if (tid == 0) {
      tau[k] = t;
      diag[k] = dk;
      sub[k] = alpha;
    }
  }
  if (i >= n) return;   // whole waves
  const double vi = sv[i], wi = sw[i];
  double s = 0.0;
  if constexpr (HELD) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int j = e * 64 + lane;
      if (j > k && j < n) {
        const double a = ai[e] - (vi * sw[j] + wi * sv[j]);
        Ai[j] = a;
        s = fma(a, sn[j], s);
      }
    }
  } else {
    for (int j = k + 1 + lane; j < n; j += 64) {
      const double a = Ai[j] - (vi * sw[j] + wi * sv[j]);
      Ai[j] = a;
      s = fma(a, sn[j], s);
    }
  }
  s = wave_sum(s);
  if (lane == 0) p_out[i] = s * scale;
}

// lam[r] = the r-th largest eigenvalue of T; norm[0] = a bound on ||T||. One
// workgroup per eigenvalue, every thread with a shift of its own.
template <int NMAX>
__global__ __launch_bounds__(kFitThreads) void fit_bisect_kernel(
    const double* __restrict__ diag, const double* __restrict__ sub, int n, int n_pca,
    double* __restrict__ lam, double* __restrict__ norm) {
  __shared__ double sd[NMAX], se2[NMAX];
  __shared__ double red[3][4];
  __shared__ int redi[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double lo = 1e308, hi = -1e308, big = 0.0;
  for (int i = tid; i < n; i += kFitThreads) {
    const double d = diag[i];
    const double el = i > 0 ? fabs(sub[i - 1]) : 0.0, er = i + 1 < n ? fabs(sub[i]) : 0.0;
    sd[i] = d;
    se2[i] = el * el;
    lo = fmin(lo, d - (el + er));
    hi = fmax(hi, d + (el + er));
    big = fmax(big, el * el);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
    big = fmax(big, __shfl_xor(big, o));
  }
  if (lane == 0) {
    red[0][wv] = lo;
    red[1][wv] = hi;
    red[2][wv] = big;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    lo = fmin(lo, red[0][w]);
    hi = fmax(hi, red[1][w]);
    big = fmax(big, red[2][w]);
  }
  const double bound = fmax(fabs(lo), fabs(hi));
  const double pivmin = 2.2250738585072014e-308 * fmax(1.0, big);
  const double slack = 4.0 * kFitEps * bound * n + 2.0 * pivmin;
  const int r = blockIdx.x;
  if (r == 0 && tid == 0) norm[0] = bound;
  const int below = n - 1 - r;   // eigenvalues smaller than the wanted one
  double a = lo - slack, b = hi + slack;
  for (int pass = 0; pass < kFitPasses; ++pass) {
    const double w = b - a;   // the same in every thread
    if (!(w > 2.0 * kFitEps * fmax(fabs(a), fabs(b)) + 2.0 * pivmin)) break;
    const double h = w * (1.0 / (kFitThreads + 1));
    const double x = a + h * double(tid + 1);
    int count = 0;
    double q = sd[0] - x;
    if (fabs(q) <= pivmin) q = -pivmin;
    count += q < 0.0;
    for (int i = 1; i < n; ++i) {
      q = (sd[i] - x) - se2[i] * fit_rcp(q);
      if (fabs(q) <= pivmin) q = -pivmin;
      count += q < 0.0;
    }
    // shifts with count <= below lie at or under the eigenvalue
    const unsigned long long under = __ballot(count <= below);
    if (lane == 0) redi[wv] = __popcll(under);
    __syncthreads();
    const int m = (redi[0] + redi[1]) + (redi[2] + redi[3]);   // count rises with the shift
    __syncthreads();
    const double na = a + h * double(m);
    if (m < kFitThreads) b = a + h * double(m + 1);
    a = m > 0 ? na : a;
  }
  if (tid == 0) lam[r] = 0.5 * (a + b);
}

// start[r] = the first index of r's cluster of close eigenvalues.
__global__ __launch_bounds__(256) void fit_clusters_kernel(const double* __restrict__ lam,
                                                           const double* __restrict__ norm,
                                                           int n_pca, int32_t* __restrict__ start,
                                                           int32_t* __restrict__ flags) {
  __shared__ int32_t s[256];
  for (int r = threadIdx.x; r < n_pca; r += 256) flags[r] = 0;   // of the panels below
  const double tol = kFitCluster * norm[0];
  int first = 0;
  for (int r0 = 0; r0 < n_pca; r0 += 256) {
    const int r = r0 + int(threadIdx.x);
    s[threadIdx.x] = r < n_pca && r > 0 && lam[r - 1] - lam[r] > tol;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int t = 0; t < 256 && r0 + t < n_pca; ++t) {
        if (s[t]) first = r0 + t;
        start[r0 + t] = first;
      }
    __syncthreads();
  }
}

// A number in [-1, 1) from two indices.
__device__ __forceinline__ double fit_noise(uint32_t i, uint32_t r) {
  uint32_t h = i * 0x9E3779B1u ^ (r + 1u) * 0x85EBCA77u;
  h = (h ^ (h >> 15)) * 0x2C1B3C6Du;
  h = (h ^ (h >> 12)) * 0x297A2D39u;
  h ^= h >> 15;
  return double(int32_t(h)) * (1.0 / 2147483648.0);
}

// Inverse iteration: row r of Z = the unit eigenvector of T for lam[r]. With
// `again` it starts from the row that is there and leaves vectors alone in
// their cluster as they are. The factors of T - x I (multiplier, the three
// diagonals of U with the main one inverted, the row swaps) and the iterate
// are in LDS, or for large n in this workgroup's 6 n doubles of `scratch`; one
// lane runs the recurrences.
template <bool LDS>
__global__ __launch_bounds__(64) void fit_vectors_kernel(
    const double* __restrict__ diag, const double* __restrict__ sub, int n, int n_pca,
    const double* __restrict__ lam, const double* __restrict__ norm,
    const int32_t* __restrict__ start, int again, double* __restrict__ scratch,
    double* __restrict__ Z) {
  __shared__ double lds[LDS ? 5 * kFitLdsN : 1];
  __shared__ uint8_t lds_swap[LDS ? kFitLdsN : 1];
  const int lane = threadIdx.x;
  double* base = LDS ? lds : scratch + int64_t(blockIdx.x) * 6 * n;
  double* u0 = base;
  double* u1 = base + n;
  double* u2 = base + 2 * n;
  double* ml = base + 3 * n;
  double* y = base + 4 * n;
  uint8_t* swapped = LDS ? lds_swap : reinterpret_cast<uint8_t*>(base + 5 * n);
  const double tiny = fmax(kFitEps * norm[0], 1e-280);
  for (int r = blockIdx.x; r < n_pca; r += gridDim.x) {
    const int first = start[r];
    const bool alone = first == r && (r + 1 >= n_pca || start[r + 1] != first);
    if (again && alone) continue;   // whole workgroups
    // equal eigenvalues of a cluster are told apart by a few roundings of T
    const double x = lam[r] - double(r - first) * kFitEps * norm[0];
    for (int i = lane; i < n; i += 64)
      y[i] = again ? Z[int64_t(r) * n + i] : fit_noise(uint32_t(i), uint32_t(r));
    if (lane == 0) {
      // (a, b, 0) is row i as the elimination left it, (c, d, e) row i + 1
      double a = diag[0] - x, b = n > 1 ? sub[0] : 0.0;
      for (int i = 0; i + 1 < n; ++i) {
        const double c = sub[i], d = diag[i + 1] - x, e = i + 2 < n ? sub[i + 1] : 0.0;
        const bool sw = fabs(c) > fabs(a);
        double piv = sw ? c : a;
        if (fabs(piv) < tiny) piv = piv < 0.0 ? -tiny : tiny;
        const double inv = fit_rcp(piv), m = (sw ? a : c) * inv;
        const double up = sw ? d : b;
        u0[i] = inv;
        u1[i] = up;
        u2[i] = sw ? e : 0.0;
        ml[i] = m;
        swapped[i] = sw;
        a = (sw ? b : d) - m * up;
        b = sw ? -m * e : e;
      }
      if (fabs(a) < tiny) a = a < 0.0 ? -tiny : tiny;
      u0[n - 1] = fit_rcp(a);
      u1[n - 1] = 0.0;
      u2[n - 1] = 0.0;
    }
    __syncthreads();
    for (int it = 0; it < (again ? 2 : 3); ++it) {
      if (lane == 0) {
        double cur = y[0];
        for (int i = 0; i + 1 < n; ++i) {
          const double next = y[i + 1];
          const bool sw = swapped[i] != 0;
          const double top = sw ? next : cur;
          y[i] = top;
          cur = (sw ? cur : next) - ml[i] * top;
        }
        double y1 = cur * u0[n - 1], y2 = 0.0;
        y[n - 1] = y1;
        for (int i = n - 2; i >= 0; --i) {
          const double v = (y[i] - u2[i] * y2 - u1[i] * y1) * u0[i];
          y[i] = v;
          y2 = y1;
          y1 = v;
        }
      }
      __syncthreads();
      double big = 0.0;
      for (int i = lane; i < n; i += 64) big = fmax(big, fabs(y[i]));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o));
      const double s = 1.0 / big;   // keeps the squares in range
      double n2 = 0.0;
      for (int i = lane; i < n; i += 64) n2 = fma(y[i] * s, y[i] * s, n2);
      const double scale = s / sqrt(wave_sum(n2));
      for (int i = lane; i < n; i += 64) y[i] *= scale;
      __syncthreads();
    }
    for (int i = lane; i < n; i += 64) Z[int64_t(r) * n + i] = y[i];
    __syncthreads();
  }
}

// Orthonormalises the rows of Z of every cluster of two or more, in order. A
// workgroup owns a panel of 16 rows. It frees them of the earlier panels of
// their cluster, panel by panel (16 x 16 coefficients and the update on FP64
// matrix cores), then of each other, and scales them to length one; all that
// twice (the second time removes what rounding left of the first). A panel is
// published when it is finished (flags[P] = epoch); a workgroup waits for panels
// with a lower index only, which are dispatched first, so the waits end. Past
// kFitWaitTicks of the 100 MHz counter it makes its rows NaN and goes on.
//
// Bound by the chain of panels: 16 dependent rows inside each, and the earlier
// panels again in the second pass. One workgroup for a cluster, row after row,
// took 748 ms for n = n_pca = 720 and rank 100 (a cluster of 620; Jacobi 112 ms),
// now 44, and 4.0 ms for 128 of 168 vectors of a decaying spectrum, now 2.2.
// LDS: the panel in LDS (n <= kFitPanelN), else in place in Z.
typedef double fit_f64x4 __attribute__((ext_vector_type(4)));
constexpr int kFitPanel = 16, kFitPanelN = 1024, kFitPanelThreads = 512;
constexpr uint64_t kFitWaitTicks = uint64_t(1) << 30;   // about 10.7 s

template <bool LDS>
__global__ __launch_bounds__(kFitPanelThreads) void fit_orthogonal_kernel(
    double* Z, int n, int n_pca, const int32_t* __restrict__ start, int32_t* flags,
    int32_t epoch) {
  constexpr int PW = kFitPanel, NT = kFitPanelThreads, NW = NT / 64;
  __shared__ double rows[LDS ? PW * (kFitPanelN + 1) : 1];
  __shared__ double part[NW][PW * PW], coef[PW * PW];
  __shared__ int32_t first[PW];   // start of each row's cluster
  __shared__ int32_t s_failed;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lt = lane >> 4;
  const int p0 = int(blockIdx.x) * PW;
  const int np = n_pca - p0 < PW ? n_pca - p0 : PW;   // rows of this panel
  bool cluster = false;
  if (lane < np) {
    const int j = p0 + lane;
    const int32_t s = start[j];
    if (wv == 0) first[lane] = s;
    cluster = s != j || (j + 1 < n_pca && start[j + 1] == s);
  }
  if (!__any(cluster)) return;   // the same in every wave
  const int ld = LDS ? (n | 1) : n;
  double* const P = LDS ? rows : Z + int64_t(p0) * n;
  if (tid == 0) s_failed = 0;
  if constexpr (LDS) {
    for (int j = wv; j < PW; j += NW)
      for (int i = lane; i < n; i += 64) P[j * ld + i] = j < np ? Z[int64_t(p0 + j) * n + i] : 0.0;
  }
  __syncthreads();
  const int C = first[0];
  int joined = 0;   // rows of the cluster that the earlier panels belong to
  while (joined < np && first[joined] == C) ++joined;
  const int groups = (n + 15) / 16;

  for (int pass = 0; pass < 2; ++pass) {
    for (int q0 = C / PW * PW; q0 < p0; q0 += PW) {
      if (pass == 0) {
        if (tid == 0) {
          const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
          while (!s_failed && __hip_atomic_load(&flags[q0 / PW], __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) < epoch) {
            if (__builtin_amdgcn_s_memrealtime() - t0 > kFitWaitTicks) s_failed = 1;
            __builtin_amdgcn_s_sleep(2);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
      }
      const double* Q = Z + int64_t(q0) * n;
      // coefficients Q P^T: slot k = lt of product e stands for column 16 u + 4 lt + e
      fit_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      const double* pj = P + (LDS || li < np ? li : np - 1) * ld;
      for (int u = wv; u < groups; u += NW) {
        double a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = 16 * u + 4 * lt + e, cc = c < n ? c : n - 1;
          a[e] = Q[int64_t(li) * n + cc];
          b[e] = pj[cc];
          if (c >= n) a[e] = b[e] = 0.0;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wv][(lt + 4 * r) * PW + li] = acc[r];
      __syncthreads();
      if (tid < PW * PW) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += part[w][tid];
        coef[tid] = q0 + tid / PW >= C && tid % PW < joined ? s : 0.0;
      }
      __syncthreads();
      for (int u = wv; u < groups; u += NW) {
        const int c = 16 * u + li, cc = c < n ? c : n - 1;
        fit_f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          d = __builtin_amdgcn_mfma_f64_16x16x4f64(coef[(4 * s + lt) * PW + li],
                                                   Q[int64_t(4 * s + lt) * n + cc], d, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (lt + 4 * r < np && c < n) P[(lt + 4 * r) * ld + c] -= d[r];
      }
      __syncthreads();
    }
    for (int j = 0; j < np; ++j) {
      const int lo = first[j] > p0 ? first[j] - p0 : 0;
      if (first[j] == p0 + j) continue;   // the first of its cluster stays as it is
      double* pj = P + j * ld;
      for (int again = 0; again < 2; ++again) {
        for (int q = lo + wv; q < j; q += NW) {
          double s = 0.0;
          for (int i = lane; i < n; i += 64) s = fma(P[q * ld + i], pj[i], s);
          s = wave_sum(s);
          if (lane == 0) coef[q] = s;
        }
        __syncthreads();
        for (int i = tid; i < n; i += NT) {
          double v = pj[i];
          for (int q = lo; q < j; ++q) v = fma(-coef[q], P[q * ld + i], v);
          pj[i] = v;
        }
        __syncthreads();
      }
      double n2 = 0.0;
      for (int i = tid; i < n; i += NT) n2 = fma(pj[i], pj[i], n2);
      n2 = wave_sum(n2);
      if (lane == 0) part[0][wv] = n2;
      __syncthreads();
      n2 = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) n2 += part[0][w];
      const double scale = 1.0 / sqrt(n2);
      for (int i = tid; i < n; i += NT) pj[i] *= scale;
      __syncthreads();
    }
  }
  if (LDS || s_failed)
    for (int j = wv; j < np; j += NW)
      for (int i = lane; i < n; i += 64)
        Z[int64_t(p0 + j) * n + i] = s_failed ? __builtin_nan("") : P[j * ld + i];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (tid == 0)
    __hip_atomic_store(&flags[blockIdx.x], epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Column r of U = H_0 H_1 ... H_{n-2} applied to row r of Z, its sign fixed by
// its entry of largest magnitude (ties: lowest row). One workgroup of WAVES
// waves per vector, 16 entries per lane in registers; the next reflector is
// loaded while the current one is applied.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void fit_back_kernel(
    const double* __restrict__ Z, const double* __restrict__ Vh, const double* __restrict__ tau,
    const double* __restrict__ lam, int n, int n_pca, float* __restrict__ U,
    double* __restrict__ sv) {
  constexpr int NT = 64 * WAVES, EPT = 16;
  __shared__ double red[2][WAVES];
  __shared__ int redi[WAVES];
  const int r = blockIdx.x, tid = threadIdx.x;
  double y[EPT], v[EPT], vn[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) y[e] = e * NT + tid < n ? Z[int64_t(r) * n + e * NT + tid] : 0.0;
  auto load = [&](double (&w)[EPT], int k) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int j = e * NT + tid;
      w[e] = j > k && j < n ? Vh[int64_t(k) * n + j] : 0.0;
    }
  };
  load(v, n - 1);
  for (int k = n - 1; k >= 0; --k) {
    if (k > 0) load(vn, k - 1);
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) s = fma(v[e], y[e], s);
    s = wave_sum(s);
    if constexpr (WAVES > 1) {
      if ((tid & 63) == 0) red[k & 1][tid >> 6] = s;
      __syncthreads();
      s = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) s += red[k & 1][w];
    }
    s *= tau[k];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      y[e] = fma(-s, v[e], y[e]);
      v[e] = vn[e];
    }
  }
  double best = -1.0, val = 0.0;
  int at = 0x7FFFFFFF;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int j = e * NT + tid;
    if (j < n && fabs(y[e]) > best) {
      best = fabs(y[e]);
      val = y[e];
      at = j;
    }
  }
  auto take = [&](double b, double w, int a) {
    if (b > best || (b == best && a < at)) {
      best = b;
      val = w;
      at = a;
    }
  };
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double b = __shfl_xor(best, o), w = __shfl_xor(val, o);
    take(b, w, __shfl_xor(at, o));
  }
  if constexpr (WAVES > 1) {
    __syncthreads();
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = best;
      red[1][tid >> 6] = val;
      redi[tid >> 6] = at;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) take(red[0][w], red[1][w], redi[w]);
  }
  const double sgn = val < 0.0 ? -1.0 : 1.0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int j = e * NT + tid;
    if (j < n) U[int64_t(j) * n_pca + r] = float(sgn * y[e]);
  }
  if (sv != nullptr && tid == 0) sv[r] = sqrt(lam[r] > 0.0 ? lam[r] : 0.0);
}

}  // namespace sorf

using namespace sorf;

// Four n x n matrices (G, later the scratch of the inverse iteration; A; the
// reflectors; the vectors of T) and a few vectors.
static size_t fit_align(size_t b) { return (b + 255) & ~size_t(255); }

constexpr int kFitScratchGroups = 64;   // workgroups of the inverse iteration outside LDS

static size_t fit_g_bytes(size_t n) {
  const size_t g = 8 * n * n, s = 8 * 6 * n * kFitScratchGroups;
  return fit_align(int(n) > kFitLdsN && s > g ? s : g);
}

size_t sorf_fit_ws_bytes(int32_t d_rep) {
  const size_t n = size_t(d_rep);
  return fit_g_bytes(n) + 3 * fit_align(8 * n * n) + 6 * fit_align(8 * n) + fit_align(8) +
         2 * fit_align(4 * n);
}

hipError_t sorf_launch_projection_fit(int64_t n_samples, int32_t d_rep, const float* sample,
                                      int32_t n_pca, float* U, double* sv, void* ws,
                                      hipStream_t st) {
  const int n = d_rep;
  char* p = static_cast<char*>(ws);
  auto part = [&](size_t bytes) {
    char* q = p;
    p += fit_align(bytes);
    return q;
  };
  const size_t mat = 8 * size_t(n) * n, vec = 8 * size_t(n);
  double* G = reinterpret_cast<double*>(part(fit_g_bytes(size_t(n))));
  double* A = reinterpret_cast<double*>(part(mat));
  double* Vh = reinterpret_cast<double*>(part(mat));
  double* Z = reinterpret_cast<double*>(part(mat));
  double* pv[2];
  pv[0] = reinterpret_cast<double*>(part(vec));
  pv[1] = reinterpret_cast<double*>(part(vec));
  double* tau = reinterpret_cast<double*>(part(vec));
  double* diag = reinterpret_cast<double*>(part(vec));
  double* sub = reinterpret_cast<double*>(part(vec));
  double* lam = reinterpret_cast<double*>(part(vec));
  double* norm = reinterpret_cast<double*>(part(8));
  int32_t* start = reinterpret_cast<int32_t*>(part(4 * size_t(n)));
  int32_t* flags = reinterpret_cast<int32_t*>(part(4 * size_t(n)));

  hipError_t err = sorf_launch_fill(reinterpret_cast<float*>(G), 2 * int64_t(n) * n, 0.0f, st);
  if (err != hipSuccess) return err;
  err = sorf_launch_gram_f64(n_samples, n, sample, nullptr, G, nullptr, st);
  if (err != hipSuccess) return err;
  const int64_t nn = int64_t(n) * n;
  hipLaunchKernelGGL(fit_init_kernel, dim3(unsigned((nn + 255) / 256)), dim3(256), 0, st, G, n, A);
  constexpr int rows = kFitThreads / 64;   // one per wave
  for (int k = 0; k < n; ++k) {
    const int left = n - 1 - k;
    const dim3 grid(unsigned(left > 0 ? (left + rows - 1) / rows : 1));
    if (n <= 1024)
      hipLaunchKernelGGL(fit_column_kernel<1024>, grid, dim3(kFitThreads), 0, st, A, n, k,
                         pv[k & 1], pv[(k + 1) & 1], Vh, tau, diag, sub);
    else
      hipLaunchKernelGGL(fit_column_kernel<4096>, grid, dim3(kFitThreads), 0, st, A, n, k,
                         pv[k & 1], pv[(k + 1) & 1], Vh, tau, diag, sub);
  }
  const dim3 each{unsigned(n_pca)};
  if (n <= 1024)
    hipLaunchKernelGGL(fit_bisect_kernel<1024>, each, dim3(kFitThreads), 0, st, diag, sub, n,
                       n_pca, lam, norm);
  else
    hipLaunchKernelGGL(fit_bisect_kernel<4096>, each, dim3(kFitThreads), 0, st, diag, sub, n,
                       n_pca, lam, norm);
  hipLaunchKernelGGL(fit_clusters_kernel, dim3(1), dim3(256), 0, st, lam, norm, n_pca, start, flags);
  // once for every vector, twice more for the vectors of clusters
  for (int round = 0; round < 3; ++round) {
    if (n <= kFitLdsN)
      hipLaunchKernelGGL(fit_vectors_kernel<true>, each, dim3(64), 0, st, diag, sub, n, n_pca,
                         lam, norm, start, int(round > 0), G, Z);
    else
      hipLaunchKernelGGL(fit_vectors_kernel<false>,
                         dim3(unsigned(n_pca < kFitScratchGroups ? n_pca : kFitScratchGroups)),
                         dim3(64), 0, st, diag, sub, n, n_pca, lam, norm, start, int(round > 0),
                         G, Z);
    const dim3 panels{unsigned((n_pca + kFitPanel - 1) / kFitPanel)}, threads{kFitPanelThreads};
    if (n <= kFitPanelN)
      hipLaunchKernelGGL(fit_orthogonal_kernel<true>, panels, threads, 0, st, Z, n, n_pca, start,
                         flags, round + 1);
    else
      hipLaunchKernelGGL(fit_orthogonal_kernel<false>, panels, threads, 0, st, Z, n, n_pca, start,
                         flags, round + 1);
  }
  if (n <= 1024)
    hipLaunchKernelGGL(fit_back_kernel<1>, each, dim3(64), 0, st, Z, Vh, tau, lam, n, n_pca, U, sv);
  else
    hipLaunchKernelGGL(fit_back_kernel<4>, each, dim3(256), 0, st, Z, Vh, tau, lam, n, n_pca, U,
                       sv);
  return hipGetLastError();
}
