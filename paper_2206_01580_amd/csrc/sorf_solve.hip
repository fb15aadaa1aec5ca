// Ridge solve (G + lambda I) alpha = Zty in FP64 on gfx950.
//
// Paper: arXiv 2206.01580, RFF subsection (regularised normal equation, solved
// by a matrix decomposition on the GPU; the matrix is symmetric positive
// definite for lambda > 0, so a Cholesky factorisation gives the paper's alpha)
// and the Training-time discussion (FP32 round-off in Z^T Z harms the
// conditioning; here the factorisation, the triangular solves and the residual
// of the iterative refinement are all FP64).
//
// Blocked right-looking Cholesky with panel width NB = 128:
//   1. factor the NB x NB diagonal block in LDS and invert it (one workgroup;
//      16 x 16 parts on FP64 MFMA, one wave on the pivots, the others beside it),
//   2. panel below: L21 = A21 L11^{-T} = A21 (L11^{-1})^T as an FP64 MFMA GEMM,
//      fused with the update of the next diagonal tile,
//   3. trailing update A22 -= L21 L21^T on the rest of the lower triangle,
//      128 x 128 tiles of FP64 MFMA.
// Triangular solves use the inverted diagonal blocks: one launch per sweep,
// one workgroup per block row, each waiting for the solved values it needs.
#include <cmath>
#include <type_traits>

#include "sorf_internal.h"

namespace sorf {

constexpr int NB = 128;
typedef double f64x4 __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ void tri_tile(int64_t t, int64_t& I, int64_t& J) {
  int64_t i = int64_t((std::sqrt(8.0 * double(t) + 1.0) - 1.0) * 0.5);
  while (i * (i + 1) / 2 > t) --i;
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  I = i;
  J = t - i * (i + 1) / 2;
}

// v_mfma_f64_16x16x4f64 operands: lane l supplies A[l%16][l/16] and B[l/16][l%16];
// the result D[l/16 + 4 r][l%16] sits in register r of lane l.
static __device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Values of the triangular sweeps' outputs are their own ready signals: a
// slot holds the signalling-NaN pattern kNotReady (never produced by
// arithmetic) until its value is stored; stores and polls are agent-scope
// atomics, so they are seen across the XCDs' L2 caches.
constexpr long long kNotReady = 0x7FF4534457454550ll;

static __device__ __forceinline__ double not_ready() { return __longlong_as_double(kNotReady); }
static __device__ __forceinline__ bool is_not_ready(double v) {
  return __double_as_longlong(v) == kNotReady;
}
static __device__ __forceinline__ double poll_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
static __device__ __forceinline__ void signal_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct SolveWs {
  double* A;     // [D][D], lower triangle used
  double* Linv;  // [nblk][NB][NB] inverses of the diagonal blocks
  double* LinvT; // [nblk][NB][NB] their transposes (row access in the forward sweep)
  double* b;     // [D]
  double* y;     // [D]
  double* dx;    // [D]
  double* part;  // [nt][nt][64] partial sums of the symmetric product
  int32_t* pflags;  // [8] strip flags of the panel kernel, [8] of syrk_next (epoch = block + 1)
};

static size_t align256(size_t n) { return (n + 255) & ~size_t(255); }

static SolveWs carve(void* ws, int32_t D) {
  const size_t nblk = (size_t(D) + NB - 1) / NB;
  char* p = static_cast<char*>(ws);
  SolveWs w;
  w.A = reinterpret_cast<double*>(p);      p += align256(sizeof(double) * size_t(D) * D);
  w.Linv = reinterpret_cast<double*>(p);   p += align256(sizeof(double) * nblk * NB * NB);
  w.LinvT = reinterpret_cast<double*>(p);  p += align256(sizeof(double) * nblk * NB * NB);
  w.b = reinterpret_cast<double*>(p);      p += align256(sizeof(double) * D);
  w.y = reinterpret_cast<double*>(p);      p += align256(sizeof(double) * D);
  w.dx = reinterpret_cast<double*>(p);     p += align256(sizeof(double) * D);
  w.part = reinterpret_cast<double*>(p);
  p += align256(sizeof(double) * ((size_t(D) + 63) / 64) * ((size_t(D) + 63) / 64) * 64);
  w.pflags = reinterpret_cast<int32_t*>(p);
  return w;
}

// A = G + lambda I on the lower triangle, promoted to FP64; clears info.
template <typename TG>
__global__ __launch_bounds__(256) void promote_kernel(const TG* __restrict__ G, int32_t D,
                                                     double lambda, double* __restrict__ A,
                                                     int32_t* __restrict__ info,
                                                     double* y, int32_t* __restrict__ pflags) {
  const int64_t i = blockIdx.y;
  const int64_t j = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i == 0 && j == 0) *info = 0;
  if (i == 0 && j < 16) pflags[j] = 0;
  if (i == 0 && j < D) signal_store(y + j, not_ready());   // output of the first forward sweep
  if (j <= i && j < D) A[i * D + j] = double(G[i * D + j]) + (i == j ? lambda : 0.0);
}

// ---------------------------------------------------------------------------
// Diagonal block: factor a 128 x 128 block in LDS and form the inverse of its
// factor.
//
// This kernel is the serial part of the factorisation: one workgroup, and the
// rest of the solve's chain waits for it. What bounds it is the length of the
// dependent chain of 128 pivots, so the block is cut into 16 x 16 parts whose
// elimination is a rank-1 update by one FP64 MFMA a pivot, without LDS or
// lane exchange: in the accumulator layout (row lane / 16 + 4 r, column
// lane % 16) row J of the symmetric part is register J / 4 of the lanes with
// lane / 16 == J % 4, which is also where the MFMA reads slot k = J % 4 of
// either operand. Wave 0 does these steps, and between two parts only the
// three products that the next part needs, all in registers; the other waves
// are one part behind it with the rest (one barrier a part). Wave 4 stays
// out of their work but for the stores, since it would take wave 0's matrix core.
// 128 x 128: 55 us with one wave on 64 x 64 halves (a column published
// through LDS a pivot, 256 steps for factor and inverse), now 26.5. A pivot
// takes 250 cycles (two MFMAs of 67, which FP64 vector instructions of the
// wave do not overlap), a part 6200 with the three products and the barrier.
//
// Row stride NB + 18 doubles: the 16 rows x 2 columns that half a wave reads
// for an MFMA operand then fall on distinct LDS banks.
// ---------------------------------------------------------------------------
constexpr int LDL = NB + 18;
constexpr int PB = 16;   // rows of a part

// 1 / d to full double precision: the hardware's estimate (within 2^-24) and one
// third-order step, which leaves its error's cube. (One Newton step left 2^-48.7;
// the exact IEEE division is a longer dependent chain on the critical path.)
static __device__ __forceinline__ double recip(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

// 1 / sqrt(d) for a positive finite d: hardware estimate plus one third-order step.
static __device__ __forceinline__ double recip_sqrt(double d) {
  const double r = __builtin_amdgcn_rsq(d);
  const double e = __builtin_fma(-d * r, r, 1.0);
  return __builtin_fma(r * e, __builtin_fma(0.375, e, 0.5), r);
}

static __device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// acc += sum_p a[row][p] b[col][p] over 16 values of p: a and b point at the
// first of 16 rows in LDS, lane (li, lt) supplies row li.
static __device__ __forceinline__ f64x4 part_nt(const double* a, const double* b, int li, int lt,
                                                f64x4 acc) {
  double av[4], bv[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    av[s] = a[li * LDL + 4 * s + lt];
    bv[s] = b[li * LDL + 4 * s + lt];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = mfma64(av[s], bv[s], acc);
  return acc;
}

// acc += sum_p a[row][p] b[p][col]: b is read along its rows.
static __device__ __forceinline__ f64x4 part_nn(const double* a, const double* b, int li, int lt,
                                                f64x4 acc) {
  double av[4], bv[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    av[s] = a[li * LDL + 4 * s + lt];
    bv[s] = b[(4 * s + lt) * LDL + li];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = mfma64(av[s], bv[s], acc);
  return acc;
}

// One wave: C is a symmetric 16 x 16 part in the accumulator layout; returns
// the inverse of its Cholesky factor (zero above the diagonal). Elimination
// of [C | I] without scaling: at pivot J, row i > J loses C[i][J] / d_J times
// row J, d_J = C[J][J]; the rows of the second half are scaled by
// 1 / sqrt(d_i) at the end. A pivot that is not positive and finite makes its
// row NaN, and the first one (of the nvalid rows inside the matrix) sets info.
static __device__ __forceinline__ f64x4 part_factor_inverse(f64x4 C, int li, int lt, int lane,
                                                            int32_t* info, int gbase,
                                                            int nvalid) {
  f64x4 X, piv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    X[r] = lt + 4 * r == li ? 1.0 : 0.0;
    piv[r] = 1.0;
  }
  double d = lane_value(C[0], 0);
  double rd = recip(d);
#pragma unroll
  for (int J = 0; J < PB; ++J) {
    const int rr = J >> 2, rq = J & 3;
    const bool own = lt == rq;
    const double row = own && li > J ? C[rr] : 0.0;   // row J = column J right of the diagonal
    const double f = -row * rd;
    const double xrow = own ? X[rr] : 0.0;
    // the next pivot, with the MFMA's own operations, beside the MFMA
    double c10 = 0.0, c11 = 0.0;
    if (J + 1 < PB) {
      c10 = lane_value(C[rr], 16 * rq + J + 1);
      c11 = lane_value(C[(J + 1) >> 2], 16 * ((J + 1) & 3) + J + 1);
    }
    if (J + 1 < PB) C = mfma64(f, row, C);
    piv[rr] = own ? d : piv[rr];
    if (J + 1 < PB) {
      d = __builtin_fma(-(c10 * rd), c10, c11);
      rd = recip(d);
    }
    X = mfma64(f, xrow, X);
  }
  int first = PB;   // row of this lane's first bad pivot
#pragma unroll
  for (int r = 3; r >= 0; --r) {
    const int i = lt + 4 * r;
    const bool bad = !(piv[r] > 0.0) || !std::isfinite(piv[r]);
    if (bad && i < nvalid) first = i;
    const double s = bad ? __builtin_nan("") : recip_sqrt(piv[r]);
    X[r] = i >= li ? X[r] * s : 0.0;
  }
  if (__any(first < PB)) {   // the rows of lane groups 0 .. 3 interleave
    int f = first;
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) f = min(f, __shfl_xor(f, o));
    if (lane == 0 && *info == 0) *info = gbase + 1 + f;
  }
  return X;
}

// Factor the diagonal block at (k, k) and write the inverse of
// L into Linv[k / NB] (the diagonal block of L itself is not needed again:
// the panel solve and the sweeps use the inverse). 512 threads. In parts,
//   X_jj = chol(A_jj)^{-1}                      A_jj updated by the parts left of it
//   L_ij = A_ij X_jj^T                          i > j
//   A_il -= L_ij L_lj^T                         j < l <= i
//   X_jc = -X_jj sum_{c <= p < j} L_jp X_pc     c < j
// Step j between two barriers: wave 0 forms L_j,j-1 and X_jj, bringing what
// they need up to date with the panels j - 2 and j - 1 itself. The helper
// waves form L_i,j-1 for i > j, apply panel j - 2 to the columns >= j, finish
// block row j - 1 of the inverse and sum the products of row j that exist.
// A helper owns the columns c of the inverse, so it waits for no other one.
// X_jc is stored in the block's upper half, at part (c, j): L_jc is still read.
__global__ __launch_bounds__(512) void potrf_diag_kernel(const double* __restrict__ A, int32_t D,
                                                        int32_t k, int32_t* __restrict__ info,
                                                        double* __restrict__ Linv) {
  __shared__ double L[NB][LDL];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lt = lane >> 4;
  const int n = (D - k) < NB ? (D - k) : NB;
  const int np = (n + PB - 1) / PB;   // parts that reach into the matrix
  // rows past the matrix are padded with the identity; every thread issues
  // its loads (columns lane and lane + 64 of the lower part, rows wv + 8 m)
  // before it stores any
  {
    const int64_t gj0 = k + min(lane, n - 1), gj1 = k + min(lane + 64, n - 1);
    double v0[16], v1[8];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const int64_t gi = k + min(wv + 8 * m, n - 1);
      v0[m] = A[gi * D + gj0];
      if (m >= 8) v1[m - 8] = A[gi * D + gj1];
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const int i = wv + 8 * m;
      L[i][lane] = (i < n && lane <= i) ? v0[m] : (i == lane ? 1.0 : 0.0);
      if (m >= 8)
        L[i][lane + 64] = (i < n && lane + 64 <= i) ? v1[m - 8] : (i == lane + 64 ? 1.0 : 0.0);
    }
  }
  __syncthreads();
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  const int helper = wv == 0 || wv == 4 ? -1 : (wv < 4 ? wv - 1 : wv - 2);   // 0 .. 5
  f64x4 S[2] = {zero, zero};   // a helper's sums of a block row of the inverse
  for (int j = 0; j <= np; ++j) {
    if (wv == 0 && j < np) {
      f64x4 C;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = lt + 4 * r;
        C[r] = L[PB * j + max(i, li)][PB * j + min(i, li)];
      }
      if (j > 0) {
        // T = (A_j,j-1)^T and then (L_j,j-1)^T = X T in the accumulator layout, whose
        // register s is what the MFMA reads as k = 4 s + lt of either operand
        f64x4 T, u = zero;
#pragma unroll
        for (int r = 0; r < 4; ++r) T[r] = L[PB * j + li][PB * (j - 1) + lt + 4 * r];
        if (j > 1) {
          const f64x4 t =
              part_nt(&L[PB * (j - 1)][PB * (j - 2)], &L[PB * j][PB * (j - 2)], li, lt, zero);
          u = part_nt(&L[PB * j][PB * (j - 2)], &L[PB * j][PB * (j - 2)], li, lt, zero);
#pragma unroll
          for (int r = 0; r < 4; ++r) T[r] -= t[r];
        }
        f64x4 P = zero;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          P = mfma64(L[PB * (j - 1) + li][PB * (j - 1) + 4 * s + lt], T[s], P);
#pragma unroll
        for (int s = 0; s < 4; ++s) u = mfma64(P[s], P[s], u);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          L[PB * j + li][PB * (j - 1) + lt + 4 * r] = P[r];
          C[r] -= u[r];
        }
      }
      C = part_factor_inverse(C, li, lt, lane, info, k + PB * j, n - PB * j);
#pragma unroll
      for (int r = 0; r < 4; ++r) L[PB * j + lt + 4 * r][PB * j + li] = C[r];
    } else if (helper >= 0 && j > 0) {
      // panel j - 1 below part (j, j - 1), and panel j - 2's update of the columns >= j
      // but for part (j, j): the parts of the lower half dealt from the last helper down
      // (with j == 1 the panel only)
      const int l1 = j == 1 ? 0 : np - 1;
      int i = j + 1, l = j - 1 + (5 - helper);
      for (;; l += 6) {
        while (i < np && l > min(i, l1)) l -= min(i, l1) - (j - 1) + 1, ++i;
        if (i >= np) break;
        if (l == j - 1) {
          f64x4 u;
#pragma unroll
          for (int r = 0; r < 4; ++r) u[r] = L[PB * i + li][PB * l + lt + 4 * r];
          if (j > 1) {
            const f64x4 w =
                part_nt(&L[PB * l][PB * (j - 2)], &L[PB * i][PB * (j - 2)], li, lt, zero);
#pragma unroll
            for (int r = 0; r < 4; ++r) u[r] -= w[r];
          }
          f64x4 P = zero;
#pragma unroll
          for (int s = 0; s < 4; ++s)
            P = mfma64(L[PB * l + li][PB * l + 4 * s + lt], u[s], P);
#pragma unroll
          for (int r = 0; r < 4; ++r) L[PB * i + li][PB * l + lt + 4 * r] = P[r];
        } else {
          const f64x4 u =
              part_nt(&L[PB * i][PB * (j - 2)], &L[PB * l][PB * (j - 2)], li, lt, zero);
#pragma unroll
          for (int r = 0; r < 4; ++r) L[PB * i + lt + 4 * r][PB * l + li] -= u[r];
        }
      }
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int c = helper + 6 * v;
        if (c < j - 1) {   // block row j - 1: the last product and the diagonal part
          S[v] = part_nn(&L[PB * (j - 1)][PB * (j - 2)], &L[PB * c][PB * (j - 2)], li, lt, S[v]);
          f64x4 x = zero;
#pragma unroll
          for (int s = 0; s < 4; ++s)
            x = mfma64(L[PB * (j - 1) + li][PB * (j - 1) + 4 * s + lt], S[v][s], x);
#pragma unroll
          for (int r = 0; r < 4; ++r) L[PB * c + lt + 4 * r][PB * (j - 1) + li] = -x[r];
        }
        S[v] = zero;
        if (j < np)        // block row j: all products but the one with L_j,j-1
          for (int p = c; p < j - 1; ++p)
            S[v] = part_nn(&L[PB * j][PB * p], &L[PB * c][PB * p], li, lt, S[v]);
      }
    }
    __syncthreads();
  }
  double* out = Linv + int64_t(k / NB) * NB * NB;
#pragma unroll 8
  for (int m = 0; m < 16; ++m) {
    const int i = wv + 8 * m;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = lane + 64 * h;
      // part (i / 16, j / 16) of the inverse, from the upper half's part (j / 16, i / 16)
      const int rj = j & ~(PB - 1), ri = i & ~(PB - 1);
      out[i * NB + j] = (i < n && j <= i) ? L[rj + i - ri][ri + j - rj] : 0.0;
    }
  }
}

// LinvT[b] = Linv[b]^T for every diagonal block (the backward sweeps read
// rows of the transposed inverses). One workgroup per block, 32 x 32 tiles
// through LDS.
__global__ __launch_bounds__(256) void transpose_blocks_kernel(const double* __restrict__ Linv,
                                                              double* __restrict__ LinvT) {
  __shared__ double t[32][33];
  const double* src = Linv + int64_t(blockIdx.x) * NB * NB;
  double* dst = LinvT + int64_t(blockIdx.x) * NB * NB;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int bi = 0; bi < NB; bi += 32)
    for (int bj = 0; bj < NB; bj += 32) {
#pragma unroll
      for (int r = 0; r < 32; r += 8) t[ty + r][tx] = src[(bi + ty + r) * NB + bj + tx];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 32; r += 8) dst[(bj + ty + r) * NB + bi + tx] = t[tx][ty + r];
      __syncthreads();
    }
}

// Trailing update A22 -= L21 L21^T on the lower triangle: tile (I, J) of the
// trailing matrix, 128 x 128, starts at block row/column k/NB + 1 + I/J.
constexpr int ST = 128;

// Strips of PR = 16 rows of the panel, the building block of the two kernels
// below. A workgroup forms its strip L_s = A_s (L_kk^{-1})^T, wave w the
// columns [16 w, +16), K = NB in 32 MFMAs straight from registers: each lane
// reads its operands from memory itself (the MFMA's slot k = lane / 16 of
// product 4 u + e stands for column 16 u + 4 (lane / 16) + e, for both
// operands: a lane reads 32 consecutive bytes, four lanes a line), and no wave reads what
// another one reads but for the 16 KB of the strip. Both products of a strip
// are so short that latency bounds them; what counts is the number of
// dependent steps. Strips of 32 rows with the inverse in LDS took 43,000
// cycles a panel: 10,000 to load, 12,700 and 11,000 for the products (with
// bank conflicts, two blocks a wave), the rest for the exchange.
constexpr int kSyrkGrid = 248;   // 8 of the 256 compute units stay free for the chain
constexpr int PR = 16;        // rows of a strip
constexpr int kStrips = NB / PR;
constexpr uint64_t kPanelWaitTicks = uint64_t(1) << 28;   // about 2.7 s
typedef double StripRows[PR][NB + 2];   // 16-byte aligned rows, 16 of them on distinct LDS banks

// Operands of one lane: row `row` of 128 columns from p (rows of A need not
// be 16-byte aligned).
static __device__ __forceinline__ void strip_operand(const double* p, int lt, double2 (&v)[16]) {
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    v[u].x = p[16 * (u >> 1) + 4 * lt + 2 * (u & 1)];
    v[u].y = p[16 * (u >> 1) + 4 * lt + 2 * (u & 1) + 1];
  }
}
static __device__ __forceinline__ f64x4 strip_product(const double2 (&a)[16],
                                                      const double2 (&b)[16]) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    acc = mfma64(a[u].x, b[u].x, acc);
    acc = mfma64(a[u].y, b[u].y, acc);
  }
  return acc;
}

// Forms the NS strips from row r0 on in A and in sP. 512 threads; ends without a barrier.
template <int NS>
static __device__ __forceinline__ void form_strips(double* __restrict__ A, int32_t D, int32_t k,
                                                   const double* __restrict__ Linv, int64_t r0,
                                                   StripRows (&sP)[NS], int wv, int li, int lt) {
  double2 a[NS][16], b[16];
#pragma unroll
  for (int j = 0; j < NS; ++j)
    strip_operand(A + min(r0 + PR * j + li, int64_t(D) - 1) * D + k, lt, a[j]);
  strip_operand(Linv + (int64_t(k / NB) * NB + 16 * wv + li) * NB, lt, b);
  // the strips are stored in place: every wave has its operands before any wave stores
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const f64x4 acc = strip_product(a[j], b);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = r0 + PR * j + lt + 4 * r;
      sP[j][lt + 4 * r][16 * wv + li] = acc[r];
      if (row < D) A[row * D + k + 16 * wv + li] = acc[r];
    }
  }
}

// A wave's 16 x 16 entries at (r0, c0), lower part inside the matrix.
static __device__ __forceinline__ void read_block(const double* __restrict__ A, int32_t D,
                                                  int64_t r0, int64_t c0, int li, int lt,
                                                  double (&c)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
    c[r] = A[min(r0 + lt + 4 * r, int64_t(D) - 1) * D + min(c0 + li, int64_t(D) - 1)];
}
static __device__ __forceinline__ void write_block(double* __restrict__ A, int32_t D, int64_t r0,
                                                   int64_t c0, int li, int lt,
                                                   const double (&c)[4], f64x4 acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t gi = r0 + lt + 4 * r, gj = c0 + li;
    if (gi < D && gi >= gj) A[gi * D + gj] = c[r] - acc[r];
  }
}

// Publishes the strips that this workgroup stored (flags = epoch).
static __device__ __forceinline__ void publish_strips(int32_t* flags, int n, int32_t epoch) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (int(threadIdx.x) < n)
    __hip_atomic_store(flags + threadIdx.x, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// One wave waits for a strip of a workgroup with a lower index, which is
// dispatched first, so the wait ends; past kPanelWaitTicks of the 100 MHz
// counter it sets *info = -1 and goes on.
static __device__ __forceinline__ void await_strip(const int32_t* flag, int32_t epoch,
                                                   int32_t* info) {
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
    if (__builtin_amdgcn_s_memrealtime() - t0 > kPanelWaitTicks) {
      int32_t expect = 0;
      __hip_atomic_compare_exchange_strong(info, &expect, -1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// Next block row of the panel, fused with the update of the next diagonal
// tile: workgroup b (0 .. 7) forms strip b of the block row below (k, k) and
// publishes it (flags[b] = epoch), then wave w <= b applies strip w to the
// 16 x 16 part (b, w) of the tile, for which it waits for that strip alone.
// The next diagonal block is therefore updated when the kernel ends, with
// the tile work spread over eight compute units. (The panel rows below the
// next block row are formed by syrk_next.) 27 us before, now 14 (21 beside
// the far update of D = 8192, which takes most of the memory path).
__global__ __launch_bounds__(512) void panel_kernel(double* __restrict__ A, int32_t D, int32_t k,
                                                   const double* __restrict__ Linv,
                                                   int32_t* __restrict__ flags,
                                                   int32_t* __restrict__ info) {
  __shared__ __attribute__((aligned(16))) StripRows sP[1];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lt = lane >> 4;
  const int b = int(blockIdx.x);
  const int32_t epoch = k / NB + 1;
  const int64_t s0 = int64_t(k) + NB, r0 = s0 + PR * b, c0 = s0 + PR * wv;
  double c[4];
  read_block(A, D, r0, c0, li, lt, c);
  form_strips<1>(A, D, k, Linv, r0, sP, wv, li, lt);
  publish_strips(flags + b, 1, epoch);
  if (wv > b) return;
  double2 av[16], bv[16];
  if (wv < b) {
    await_strip(flags + wv, epoch, info);
    strip_operand(A + min(c0 + li, int64_t(D) - 1) * D + k, lt, bv);
  } else {
    strip_operand(sP[0][li], lt, bv);
  }
  strip_operand(sP[0][li], lt, av);
  write_block(A, D, r0, c0, li, lt, c, strip_product(av, bv));
}

// The part of the trailing update that the next panel reads, fused with the
// panel rows it needs. Tiles of the trailing matrix's first block column
// below its diagonal, (I, 0) for I >= 1, each in kStrips / NS workgroups: a
// workgroup forms NS strips of L_I and updates its rows of the tile with
// C -= L_I L_0^T, L_0 being the next block row that the chain's panel kernel
// wrote. The last kStrips workgroups update the diagonal tile (1, 1) of the
// block after next (the tile (0, 0) is updated by the panel kernel) once the
// workgroups of tile (1, 0) have published L_1 (flags[8 + h] = epoch).
// NS = 1 while every compute unit takes one workgroup, the shortest chain;
// above that 2, since a workgroup reads the 256 KB of L_kk^{-1} and L_0
// whatever its number of strips (63 tiles: 32 us against 39 with NS = 1).
// Tiles in four parts of 32 rows with operands through LDS took 19.5 us at
// D = 1000, now 17; at D = 8192 24 on average against 22, the price of one
// shape for the short steps, where the chain waits for this kernel.
template <int NS>
__global__ __launch_bounds__(512) void syrk_next_kernel(double* __restrict__ A, int32_t D,
                                                       int32_t k, int32_t nt,
                                                       const double* __restrict__ Linv,
                                                       int32_t* __restrict__ flags,
                                                       int32_t* __restrict__ info) {
  __shared__ __attribute__((aligned(16))) StripRows sP[NS];
  constexpr int kParts = kStrips / NS;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lt = lane >> 4;
  const int n_first = (nt - 1) * kParts;   // workgroups of the first block column
  const int32_t epoch = k / NB + 1;
  const int64_t s0 = int64_t(k) + NB;
  double c[NS][4];
  double2 av[16], bv[16];
  if (int(blockIdx.x) >= n_first) {   // diagonal tile (1, 1)
    const int h = int(blockIdx.x) - n_first;
    if (wv > h) return;
    const int64_t r0 = s0 + NB + PR * h, c0 = s0 + NB + PR * wv;
    if (r0 >= D) return;
    read_block(A, D, r0, c0, li, lt, c[0]);
    await_strip(flags + 8 + h, epoch, info);
    strip_operand(A + min(r0 + li, int64_t(D) - 1) * D + k, lt, av);
    if (wv < h) await_strip(flags + 8 + wv, epoch, info);
    strip_operand(A + min(c0 + li, int64_t(D) - 1) * D + k, lt, bv);
    write_block(A, D, r0, c0, li, lt, c[0], strip_product(av, bv));
    return;
  }
  const int64_t t = blockIdx.x / kParts;
  const int h = int(blockIdx.x % kParts) * NS;
  const int64_t r0 = s0 + ST * (t + 1) + PR * h, c0 = s0 + PR * wv;
  if (r0 >= D) return;   // nobody waits for a strip past the matrix
#pragma unroll
  for (int j = 0; j < NS; ++j) read_block(A, D, r0 + PR * j, c0, li, lt, c[j]);
  form_strips<NS>(A, D, k, Linv, r0, sP, wv, li, lt);
  if (t == 0)
    publish_strips(flags + 8 + h, NS, epoch);
  else
    __syncthreads();
  strip_operand(A + (c0 + li) * D + k, lt, bv);
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    strip_operand(sP[j][li], lt, av);
    write_block(A, D, r0 + PR * j, c0, li, lt, c[j], strip_product(av, bv));
  }
}

// The rest of the trailing update, tiles (I, J) with 1 <= J <= I other than
// (1, 1). The grid of at most kSyrkGrid workgroups stays below the number of
// compute units so that the panel and diagonal kernels of the next steps find
// free units while it runs.
//
// A workgroup takes an equal run of the units of 128 rows x 32 columns, in
// row-major order. Its eight waves keep their 16 panel rows for all of
// K = NB in registers (64 of them) while the run stays in one block row, and
// the 32 rows of L_J of one unit after the other come through a ring of
// kFarRing LDS slots, copied there without registers, kFarRing - 1 units
// ahead, with one barrier a unit. The entries of the unit are read one unit
// ahead and written when it ends.
// Bound by the FP64 matrix cores (4 us a unit at 64 to 67 cycles an MFMA),
// next by the entries' own traffic (64 KB read and written a unit, 2.3 ms of
// a solve of D = 8192 at the rate of a copy), which this order spreads
// evenly: in whole tiles of 128 x 128 every workgroup's 128 KB came and went
// in the same moment and the matrix cores waited for it. Whole lines of L_J
// are copied (1 KB a row); 64 consecutive bytes a lane through registers
// touched 64 cache lines a load. Runs of units leave no round of tiles nearly
// empty. Sum over a solve of D = 8192: 5.6 ms with tiles through registers,
// 4.6 with tiles through LDS copies, now 3.9 (4.3 when every unit also waited
// for the copies in flight).
//
// In an LDS row, pair p of columns sits at p ^ (row % 16): the 16 rows that a
// group of lanes reads fall on distinct banks, without padding, which a
// 16-byte copy cannot leave. The MFMA's slot k = lane / 16 of product 2 u + e
// stands for column 8 u + 2 (lane / 16) + e, for both operands.
// EVEN: rows of A are 16-byte aligned; else 4-byte copies, four times as many.
constexpr int kFarCols = 32, kFarRing = 4;
static __device__ __forceinline__ double& at(double* base, uint32_t bytes) {
  return *reinterpret_cast<double*>(reinterpret_cast<char*>(base) + bytes);
}
static __device__ __forceinline__ void dma16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
static __device__ __forceinline__ void dma4(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)lds, 4, 0, 0);
}

// Unit q of block row r of the sub-triangle from tile (1, 1): rows
// k + NB + ST (r + 1) .., columns k + NB + ST + kFarCols q ..
struct FarUnit {
  int64_t r, q;
  static constexpr int64_t kPerTile = ST / kFarCols;
  __device__ void set(int64_t u) {   // kPerTile r (r + 1) / 2 units before row r
    int64_t I, J;
    tri_tile(u / kPerTile, I, J);
    r = I;
    q = J * kPerTile + u % kPerTile;
  }
  __device__ void next() {
    if (++q == kPerTile * (r + 1)) {
      q = 0;
      ++r;
    }
  }
};

template <bool EVEN>
__global__ __launch_bounds__(512) void syrk_far_kernel(double* __restrict__ A, int32_t D,
                                                      int32_t k, int64_t n_sub) {
  constexpr int kRow = NB * 8, kSlot = kFarCols * kRow;   // bytes
  constexpr int kAhead = kFarRing - 1;
  __shared__ __attribute__((aligned(16))) char ring[kFarRing][kSlot];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lt = lane >> 4;
  const int64_t s0 = int64_t(k) + NB + ST;
  // the workgroups of an XCD (b % 8) take neighbouring runs
  const int64_t G = gridDim.x, x = blockIdx.x & 7;
  const int64_t w = x * (G / 8) + min(x, G % 8) + blockIdx.x / 8;
  const int64_t n_units = (n_sub - 1) * FarUnit::kPerTile;   // all but tile (1, 1), the first
  const int64_t u0 = n_units * w / G;
  const int n = int(n_units * (w + 1) / G - u0);
  if (n == 0) return;
  FarUnit cur, ahead, copied;
  cur.set(u0 + FarUnit::kPerTile);
  ahead = copied = cur;

  // rows 4 wv .. + 3 of a unit's slot; rows past the matrix repeat its last
  // one: they only reach entries that are not stored
  uint32_t oS[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int sw = (4 * wv + i) & 15;
    oS[i] = EVEN ? uint32_t(lane ^ sw) * 16u : uint32_t((lane >> 2) ^ sw) * 16u + (lane & 3) * 4u;
  }
  // every unit starts one copy and one read of entries, past the last unit
  // those of the last one again: the waits below count on it
  int left = n - 1;   // units after `copied`
  const auto copy = [&](int slot) {
    const int64_t col0 = s0 + kFarCols * copied.q + 4 * wv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double* src = A + min(col0 + i, int64_t(D) - 1) * D + k;
      char* dst = ring[slot] + (4 * wv + i) * kRow;
      if constexpr (EVEN) {
        dma16(&at(src, oS[i]), dst);
      } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) dma4(&at(src, oS[i] + 256u * p), dst + 256 * p);
      }
    }
    if (left > 0) copied.next();
    --left;
  };
  // copies and reads of entries (not the stores) issued after a unit's copies
  // until its barrier, with kAhead == 3
  constexpr int kLater = 3 * 8 + 2 * (EVEN ? 4 : 16);
  static_assert(kAhead == 3 && kLater < 64, "vmcnt range");

  double2 ar[16];
  const auto load_rows = [&]() {
    const int64_t row = min(s0 + ST * cur.r + 16 * wv + li, int64_t(D) - 1);
    const double* src = A + row * D + k + 2 * lt;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if constexpr (EVEN) {
        ar[u] = *reinterpret_cast<const double2*>(src + 8 * u);
      } else {
        ar[u].x = src[8 * u];
        ar[u].y = src[8 * u + 1];
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0) here, or every unit waits for its successor's loads
  };
  double c0[2][4], c1[2][4];
  const auto load_entries = [&](const FarUnit& f, double (&v)[2][4]) {
    const int64_t I0 = s0 + ST * f.r, J0 = s0 + kFarCols * f.q;
    double* pC = A + I0 * D;
    const int last = int(min(D - I0, int64_t(ST))) - 1;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t o = uint32_t(min(16 * wv + lt + 4 * r, last)) * uint32_t(D) * 8u;
#pragma unroll
      for (int b = 0; b < 2; ++b)
        v[b][r] = at(pC, o + uint32_t(min(J0 + 16 * b + li, int64_t(D) - 1)) * 8u);
    }
  };

#pragma unroll
  for (int s = 0; s < kAhead; ++s) copy(s);
  load_rows();
  load_entries(cur, c0);
  const uint32_t read0 = uint32_t(li * kRow + 16 * (lt ^ li));
  // SLOT = s % kFarRing as a constant. (The operands are read as 8-byte pairs,
  // which become 16-byte reads: read as double2 the compiler makes each wait for
  // every copy in flight, whatever its slot.)
  const auto unit = [&](int s, auto kSlotOf, double (&c)[2][4], double (&cn)[2][4]) {
    constexpr int SLOT = decltype(kSlotOf)::value;
    // this wave's copies for the unit have landed; behind the barrier every
    // wave's have, and every wave has read the slot that is filled next
    if (s >= 2)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLater) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    copy((SLOT + kAhead) % kFarRing);
    asm volatile("" ::: "memory");   // kLater counts the reads below as issued after the copies
    if (s + 1 < n) ahead.next();
    load_entries(ahead, cn);   // of the last unit again, at the end
    const int64_t I0 = s0 + ST * cur.r, J0 = s0 + kFarCols * cur.q;
    const int64_t below = I0 + 16 * wv - J0;   // the wave's first row against the unit's first column
    f64x4 acc[2];
    acc[0] = acc[1] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (below + 15 >= 0) {   // not above the diagonal
      const char* slot = ring[SLOT];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const char* p = slot + (read0 ^ uint32_t(64 * u));
        const double* q0 = reinterpret_cast<const double*>(p);
        const double* q1 = reinterpret_cast<const double*>(p + 16 * kRow);
        const double2 b0 = make_double2(q0[0], q0[1]), b1 = make_double2(q1[0], q1[1]);
        acc[0] = mfma64(ar[u].x, b0.x, acc[0]);
        acc[1] = mfma64(ar[u].x, b1.x, acc[1]);
        acc[0] = mfma64(ar[u].y, b0.y, acc[0]);
        acc[1] = mfma64(ar[u].y, b1.y, acc[1]);
      }
      // vmcnt(12) with 16-byte copies, (24) without: c's reads are older than this
      // unit's copies and reads, which the compiler would also wait for
      __builtin_amdgcn_s_waitcnt(EVEN ? 0x0f7c : 0x4f78);
      double* pC = A + I0 * D;
      const uint32_t o = uint32_t(16 * wv + lt) * uint32_t(D) * 8u + uint32_t(J0 + li) * 8u;
      if (below >= kFarCols - 1 && I0 + ST <= D) {   // strictly below the diagonal, inside the matrix
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            at(pC, o + uint32_t(4 * r) * uint32_t(D) * 8u + 128u * b) = c[b][r] - acc[b][r];
      } else {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (I0 + 16 * wv + lt + 4 * r < D && below + lt + 4 * r >= 16 * b + li)
              at(pC, o + uint32_t(4 * r) * uint32_t(D) * 8u + 128u * b) = c[b][r] - acc[b][r];
      }
    }
    const int64_t row = cur.r;
    cur.next();
    if (cur.r != row && s + 1 < n) load_rows();
  };
  static_assert(kFarRing == 4, "units in turn");
  for (int s = 0; s < n; s += 4) {   // the entries' registers change places, not values
    unit(s, std::integral_constant<int, 0>(), c0, c1);
    if (s + 1 < n) unit(s + 1, std::integral_constant<int, 1>(), c1, c0);
    if (s + 2 < n) unit(s + 2, std::integral_constant<int, 2>(), c0, c1);
    if (s + 3 < n) unit(s + 3, std::integral_constant<int, 3>(), c1, c0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy outlives the workgroup's LDS
}

// ---------------------------------------------------------------------------
// Triangular sweeps: one launch per sweep, one workgroup (512 threads) per
// block row, in dependency order: a workgroup only waits for blocks owned by
// workgroups with a lower index, which are dispatched before it, so the
// waits always end. Every solved value is its own ready signal: the output
// vectors hold a signalling-NaN pattern (kNotReady, which arithmetic never
// produces) until the value is stored, and consumers poll the values they
// need with agent-scope atomic loads, each wave on its own (no workgroup
// barrier and no separate flag round trip on the dependency chain). Loads of
// L that do not depend on the awaited block are issued before the wait. A
// wait that exceeds kSweepWaitTicks of the 100 MHz real-time counter sets
// *info = -1 (when it is still 0) and stops waiting in that wave, so every
// wave exits. The forward sweep marks its output of the backward sweep not
// ready; the backward sweep marks each block of its input not ready once it
// has read it, ready for the next forward sweep; the promote kernel marks
// the forward output not ready at the start of a solve.
constexpr uint64_t kSweepWaitTicks = uint64_t(1) << 28;   // about 2.7 s

// Re-polls until no lane of the wave holds a not-ready value (or the wait
// times out); v[] are the values at p[], reloaded where still not ready.
template <int N>
static __device__ __forceinline__ void wave_wait(const double* const (&p)[N], double (&v)[N],
                                                 int32_t* info, bool& failed) {
  bool pending = false;
#pragma unroll
  for (int t = 0; t < N; ++t) pending |= is_not_ready(v[t]);
  if (!__any(pending) || failed) return;
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  while (true) {
    __builtin_amdgcn_s_sleep(1);
    pending = false;
#pragma unroll
    for (int t = 0; t < N; ++t) {
      if (is_not_ready(v[t])) v[t] = poll_load(p[t]);
      pending |= is_not_ready(v[t]);
    }
    if (!__any(pending)) return;
    if (__builtin_amdgcn_s_memrealtime() - t0 > kSweepWaitTicks) {
      if ((threadIdx.x & 63) == 0) {
        int32_t expect = 0;
        __hip_atomic_compare_exchange_strong(info, &expect, -1, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      failed = true;
      return;
    }
  }
}

// Sums 16 per-lane partials over the 64 lanes of a wave: afterwards every
// lane with (lane >> 2) & 15 == r holds the full sum of partial r.
static __device__ __forceinline__ double wave_sum16(double (&p)[16], int lane) {
#pragma unroll
  for (int lvl = 0; lvl < 4; ++lvl) {
    const int mask = 32 >> lvl, half = 8 >> lvl;
    const bool upper = (lane & mask) != 0;
#pragma unroll
    for (int r = 0; r < half; ++r) {
      const double keep = upper ? p[r + half] : p[r];
      const double send = upper ? p[r] : p[r + half];
      p[r] = keep + __shfl_xor(send, mask);
    }
  }
  const double t = p[0] + __shfl_xor(p[0], 2);
  return t + __shfl_xor(t, 1);
}

// out[i] = sum_c M[c][i] v[c] for a 128 x 128 block stored row-major (c rows);
// thread (i, q) holds M[32 q + m][i], m < 32, and the four quarters are added
// in a fixed order. v and red are LDS; red holds 4 x 128 doubles. The results
// are stored as ready signals.
static __device__ __forceinline__ void block_mvT_load(const double* __restrict__ M, double (&a)[32],
                                                      int tid) {
  const int i = tid & 127, q = tid >> 7;
#pragma unroll
  for (int m = 0; m < 32; ++m) a[m] = M[(32 * q + m) * NB + i];
}
static __device__ __forceinline__ void block_mvT_finish(const double (&a)[32], const double* v,
                                                        int n, double* out, double (*red)[NB],
                                                        int tid) {
  const int i = tid & 127, q = tid >> 7;
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int m = 0; m < 32; m += 2) {
    s0 = __builtin_fma(a[m], v[32 * q + m], s0);
    s1 = __builtin_fma(a[m + 1], v[32 * q + m + 1], s1);
  }
  red[q][i] = s0 + s1;
  __syncthreads();
  if (q == 0 && i < n) signal_store(out + i, (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]));
}

// Forward sweep L y = b, left-looking by block rows:
//   y_k = L_kk^{-1} (b_k - sum_{j<k} L_kj y_j).
// Workgroup k: wave w owns rows 16 w .. 16 w + 15 of the block; lane l holds
// columns l and l + 64 of each block L_kj (coalesced 512-byte row reads) and
// keeps per-lane partial sums over all j, reduced across lanes once. y must
// be not ready on entry; x (the backward sweep's output) is marked not ready.
__global__ __launch_bounds__(512) void sweep_fwd_kernel(const double* __restrict__ A,
                                                       const double* __restrict__ LinvT, int32_t D,
                                                       const double* __restrict__ b, double* y,
                                                       double* x, int32_t* __restrict__ info) {
  __shared__ double rv[NB];
  __shared__ double red[4][NB];
  bool failed = false;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int k = blockIdx.x;
  const int64_t r0 = int64_t(k) * NB;
  const int n = (D - r0) < NB ? int(D - r0) : NB;
  if (tid < n) signal_store(x + r0 + tid, not_ready());
  double inv[32];
  block_mvT_load(LinvT + int64_t(k) * NB * NB, inv, tid);
  double acc[16][2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r][0] = acc[r][1] = 0.0;
  for (int j = 0; j < k; ++j) {
    double lb[16][2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = r0 + 16 * wv + r;
      const double* p = A + (row < D ? row : D - 1) * D + int64_t(j) * NB;
      lb[r][0] = p[lane];
      lb[r][1] = p[lane + 64];
    }
    const double* const yp[2] = {y + int64_t(j) * NB + lane, y + int64_t(j) * NB + 64 + lane};
    double yv[2] = {poll_load(yp[0]), poll_load(yp[1])};
    wave_wait<2>(yp, yv, info, failed);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[r][0] = __builtin_fma(lb[r][0], yv[0], acc[r][0]);
      acc[r][1] = __builtin_fma(lb[r][1], yv[1], acc[r][1]);
    }
  }
  double ps[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) ps[r] = acc[r][0] + acc[r][1];
  const double s = wave_sum16(ps, lane);
  if ((lane & 3) == 0) {
    const int i = 16 * wv + ((lane >> 2) & 15);
    rv[i] = i < n ? b[r0 + i] - s : 0.0;
  }
  __syncthreads();
  block_mvT_finish(inv, rv, n, y + r0, red, tid);
}

// Backward sweep L^T x = y, by block rows of L^T from the last:
//   x_k = L_kk^{-T} (y_k - sum_{j>k} L_jk^T x_j).
// Workgroup g owns block k = nblk - 1 - g. Thread (c, q) holds column c of
// the block and rows 32 q .. 32 q + 31 of each block L_jk (coalesced over c),
// so the products need no cross-lane sums; the quarters are added once.
// Lane m < 32 of a wave polls x_j[32 q + m]; the values reach the other
// lanes by shuffles. x must be not ready on entry; y_k is marked not ready
// after it is read.
__global__ __launch_bounds__(512) void sweep_bwd_kernel(const double* __restrict__ A,
                                                       const double* __restrict__ Linv, int32_t D,
                                                       double* y, double* x,
                                                       int32_t* __restrict__ info) {
  __shared__ double rv[NB];
  __shared__ double red[4][NB];
  bool failed = false;
  const int tid = threadIdx.x, lane = tid & 63;
  const int c = tid & 127, q = tid >> 7;
  const int nblk = (D + NB - 1) / NB;
  const int k = nblk - 1 - int(blockIdx.x);
  const int64_t c0 = int64_t(k) * NB;
  const int n = (D - c0) < NB ? int(D - c0) : NB;
  double inv[32];
  block_mvT_load(Linv + int64_t(k) * NB * NB, inv, tid);
  const int64_t col = c0 + (c < n ? c : n - 1);
  double acc = 0.0;
  for (int j = nblk - 1; j > k; --j) {
    const int64_t rj = int64_t(j) * NB + 32 * q;
    double lb[32];
#pragma unroll
    for (int m = 0; m < 32; ++m) {
      const int64_t row = rj + m;
      lb[m] = row < D ? A[row * D + col] : 0.0;
    }
    const int64_t mine = rj + (lane & 31);
    const double* const xp[1] = {x + (mine < D ? mine : D - 1)};
    double xv[1] = {poll_load(xp[0])};
    wave_wait<1>(xp, xv, info, failed);
#pragma unroll
    for (int m = 0; m < 32; ++m) acc = __builtin_fma(lb[m], __shfl(xv[0], m), acc);
  }
  red[q][c] = acc;
  __syncthreads();
  if (q == 0 && c < n) {
    rv[c] = y[c0 + c] - ((red[0][c] + red[1][c]) + (red[2][c] + red[3][c]));
    signal_store(y + c0 + c, not_ready());   // for the next forward sweep
  } else if (q == 0) {
    rv[c] = 0.0;
  }
  __syncthreads();
  block_mvT_finish(inv, rv, n, x + c0, red, tid);
}

// Partial sums of (lower-stored symmetric G) x over 64 x 64 tiles:
// part[X][Y][.] = contribution to rows of block X from the tile pairing X and Y.
// Thread t holds 4 x 4 entries of the tile (rows t / 16 + 16 m, columns
// 4 (t % 16) + c); row sums reduce over the 16 lanes of a row group, column
// sums over the 4 row groups of a wave and then the 4 waves, all in a fixed
// order.
template <typename TG>
__global__ __launch_bounds__(256) void symv_tiles_kernel(const TG* __restrict__ G, int32_t D,
                                                        const double* __restrict__ x,
                                                        double* __restrict__ part) {
  __shared__ double csum[4][64];
  __shared__ double rsum[64];
  int64_t I, J;
  tri_tile(blockIdx.x, I, J);
  const int64_t nt = (int64_t(D) + 63) / 64;
  const int64_t I0 = I * 64, J0 = J * 64;
  const bool diag = I == J;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c0 = 4 * (tid & 15), r0 = tid >> 4;   // rows r0 + 16 m
  double g[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int64_t gi = I0 + r0 + 16 * m;
    const int64_t gic = gi < D ? gi : int64_t(D) - 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t gj = J0 + c0 + c;
      const TG v = G[gic * D + (gj < D ? gj : int64_t(D) - 1)];
      g[m][c] = (gi < D && gj < D && gj <= gi) ? double(v) : 0.0;
    }
  }
  double xj[4], xi[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) xj[c] = J0 + c0 + c < D ? x[J0 + c0 + c] : 0.0;
#pragma unroll
  for (int m = 0; m < 4; ++m) xi[m] = I0 + r0 + 16 * m < D ? x[I0 + r0 + 16 * m] : 0.0;
  // rows: G x over this tile's columns; columns: G^T x over its rows (strictly
  // below the diagonal on a diagonal tile, where the row sums already hold it)
  double rs[4], cs[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) rs[m] = ((g[m][0] * xj[0] + g[m][1] * xj[1]) + g[m][2] * xj[2]) + g[m][3] * xj[3];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cs[c] = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bool strict = !diag || (r0 + 16 * m > c0 + c);
      cs[c] += strict ? g[m][c] * xi[m] : 0.0;
    }
  }
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) rs[m] += __shfl_xor(rs[m], o);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cs[c] += __shfl_xor(cs[c], 16);
    cs[c] += __shfl_xor(cs[c], 32);
  }
  if ((tid & 15) == 0) {
#pragma unroll
    for (int m = 0; m < 4; ++m) rsum[r0 + 16 * m] = rs[m];
  }
  if (lane < 16) {
#pragma unroll
    for (int c = 0; c < 4; ++c) csum[wv][c0 + c] = cs[c];
  }
  __syncthreads();
  if (tid < 64) {
    const double col = (csum[0][tid] + csum[1][tid]) + (csum[2][tid] + csum[3][tid]);
    if (diag) {
      part[(I * nt + I) * 64 + tid] = rsum[tid] + col;
    } else {
      part[(I * nt + J) * 64 + tid] = rsum[tid];
      part[(J * nt + I) * 64 + tid] = col;
    }
  }
}

// r = Zty - lambda x - sum_Y part[X][Y]: one workgroup per 64-row block X;
// thread (i, q) sums Y in [q nt / 4, (q + 1) nt / 4) in order and the four
// quarters are added in a fixed order.
template <typename TG>
__global__ __launch_bounds__(256) void residual_kernel(const double* __restrict__ part, int32_t D,
                                                      double lambda, const TG* __restrict__ rhs,
                                                      const double* __restrict__ x,
                                                      double* __restrict__ r) {
  __shared__ double qs[4][64];
  const int64_t nt = (int64_t(D) + 63) / 64;
  const int64_t X = blockIdx.x;
  const int i = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int64_t y0 = nt * q / 4, y1 = nt * (q + 1) / 4;
  double s = 0.0;
  for (int64_t Y = y0; Y < y1; ++Y) s += part[(X * nt + Y) * 64 + i];
  qs[q][i] = s;
  __syncthreads();
  const int64_t gi = X * 64 + i;
  if (q == 0 && gi < D)
    r[gi] = (double(rhs[gi]) - lambda * x[gi]) - ((qs[0][i] + qs[1][i]) + (qs[2][i] + qs[3][i]));
}

template <typename TG>
__global__ void to_double_kernel(const TG* __restrict__ a, double* __restrict__ b, int32_t n) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) b[i] = double(a[i]);
}

__global__ void axpy_kernel(double* __restrict__ x, const double* __restrict__ d, int32_t n) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) x[i] += d[i];
}

static hipError_t solve_triangular(const SolveWs& w, int32_t D, const double* rhs, double* tmp,
                                   double* out, int32_t* info, hipStream_t st) {
  // L tmp = rhs, then L^T out = tmp: one launch per sweep, one workgroup per block
  const unsigned nblk = unsigned((D + NB - 1) / NB);
  hipLaunchKernelGGL(sweep_fwd_kernel, dim3(nblk), dim3(512), 0, st, w.A, w.LinvT, D, rhs, tmp,
                     out, info);
  hipLaunchKernelGGL(sweep_bwd_kernel, dim3(nblk), dim3(512), 0, st, w.A, w.Linv, D, tmp, out,
                     info);
  return hipGetLastError();
}

template <typename TG>
static hipError_t launch_solve(int32_t D, const TG* G, const TG* Zty, double lambda,
                               int32_t n_refine, double* alpha, int32_t* info, void* ws,
                               hipStream_t st, hipStream_t side, hipEvent_t ev_panel,
                               hipEvent_t ev_next) {
  const SolveWs w = carve(ws, D);
  const unsigned vg = unsigned((D + 255) / 256);
  hipLaunchKernelGGL(promote_kernel<TG>, dim3(vg, unsigned(D)), dim3(256), 0, st, G, D, lambda,
                     w.A, info, w.y, w.pflags);
  // Right-looking blocked Cholesky with lookahead over two streams. Caller's
  // stream (the chain of dependent steps): the panel rows of the next block
  // row, fused with the update of the next diagonal tile (8 workgroups), then
  // the factorisation of that block. Second stream: the other panel rows, the
  // trailing tiles the next panel reads (first block column and the next
  // diagonal tile but one), then the rest of the trailing update in a
  // persistent grid that leaves compute units free, so the chain's kernels of
  // the following steps run beside it. The chain waits for the next-panel
  // tiles through an event. Every tile is updated by the steps in order: the
  // second stream runs the far update of step k before the next-panel tiles
  // of step k + 1. Only stream events order kernels of different streams, so
  // the schedule stays correct when a tool serialises the launches.
  // The second stream and both events belong to the caller. Without them
  // (side == nullptr) every launch goes to the caller's stream in the same
  // order, which serialises the chain behind each trailing update but runs
  // the same kernels on the same data: the result is bitwise the same.
  const bool two = side != nullptr;
  if (!two) side = st;
  hipError_t e = hipSuccess;
  hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(512), 0, st, w.A, D, 0, info, w.Linv);
  for (int32_t k = 0; k + NB < D; k += NB) {
    const int64_t rest = int64_t(D) - k - NB;
    const int64_t nt = (rest + 127) / 128;
    const int64_t nwg = (rest + PR - 1) / PR;
    const int64_t strips = nwg < NB / PR ? nwg : NB / PR;
    hipLaunchKernelGGL(panel_kernel, dim3(unsigned(strips)), dim3(512), 0, st, w.A, D, k, w.Linv,
                       w.pflags, info);
    // rows below the next block row (nt > 1): their panel rows are formed by
    // syrk_next together with the tiles that read them
    const bool side_work = nt > 1;
    if (side_work) {
      if (two) {
        if ((e = hipEventRecord(ev_panel, st)) != hipSuccess) return e;
        if ((e = hipStreamWaitEvent(side, ev_panel, 0)) != hipSuccess) return e;
      }
      const bool one = (nt - 1) * kStrips <= 256;   // strips against compute units
      const int64_t parts = (nt - 1) * (one ? kStrips : kStrips / 2) + kStrips;
      if (one)
        hipLaunchKernelGGL(syrk_next_kernel<1>, dim3(unsigned(parts)), dim3(512), 0, side, w.A, D,
                           k, int32_t(nt), w.Linv, w.pflags, info);
      else
        hipLaunchKernelGGL(syrk_next_kernel<2>, dim3(unsigned(parts)), dim3(512), 0, side, w.A, D,
                           k, int32_t(nt), w.Linv, w.pflags, info);
      if (two && (e = hipEventRecord(ev_next, side)) != hipSuccess) return e;
      const int64_t n_sub = (nt - 1) * nt / 2;   // sub-triangle from (1, 1)
      if (n_sub > 1) {
        const int64_t units = (n_sub - 1) * FarUnit::kPerTile;
        const int64_t g = units < kSyrkGrid ? units : kSyrkGrid;
        if (D % 2 == 0)
          hipLaunchKernelGGL(syrk_far_kernel<true>, dim3(unsigned(g)), dim3(512), 0, side, w.A, D,
                             k, n_sub);
        else
          hipLaunchKernelGGL(syrk_far_kernel<false>, dim3(unsigned(g)), dim3(512), 0, side, w.A, D,
                             k, n_sub);
      }
    }
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(512), 0, st, w.A, D, k + NB, info,
                       w.Linv);
    if (two && side_work && (e = hipStreamWaitEvent(st, ev_next, 0)) != hipSuccess) return e;
  }
  // the last far update (if any) before the sweeps read L
  if (two) {
    if ((e = hipEventRecord(ev_next, side)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(st, ev_next, 0)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(transpose_blocks_kernel, dim3(unsigned((D + NB - 1) / NB)), dim3(256), 0, st,
                     w.Linv, w.LinvT);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(to_double_kernel<TG>, dim3(vg), dim3(256), 0, st, Zty, w.b, D);
  e = solve_triangular(w, D, w.b, w.y, alpha, info, st);
  if (e != hipSuccess) return e;
  const int64_t nt = (int64_t(D) + 63) / 64;
  for (int32_t it = 0; it < n_refine; ++it) {
    hipLaunchKernelGGL(symv_tiles_kernel<TG>, dim3(unsigned(nt * (nt + 1) / 2)), dim3(256), 0, st,
                       G, D, alpha, w.part);
    hipLaunchKernelGGL(residual_kernel<TG>, dim3(unsigned(nt)), dim3(256), 0, st, w.part, D,
                       lambda, Zty, alpha, w.b);
    e = solve_triangular(w, D, w.b, w.y, w.dx, info, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(axpy_kernel, dim3(vg), dim3(256), 0, st, alpha, w.dx, D);
  }
  return hipGetLastError();
}

}  // namespace sorf

using namespace sorf;

size_t sorf_solve_ws_bytes(int32_t D) {
  const size_t nblk = (size_t(D) + NB - 1) / NB;
  const size_t nt = (size_t(D) + 63) / 64;
  return align256(sizeof(double) * size_t(D) * D) + 2 * align256(sizeof(double) * nblk * NB * NB) +
         3 * align256(sizeof(double) * D) + align256(sizeof(double) * nt * nt * 64) + 256;
}

hipError_t sorf_launch_solve(int32_t D, const float* G, const float* Zty, double lambda,
                             int32_t n_refine, double* alpha, int32_t* info, void* ws,
                             hipStream_t st, hipStream_t side, hipEvent_t ev_fork,
                             hipEvent_t ev_join) {
  return launch_solve<float>(D, G, Zty, lambda, n_refine, alpha, info, ws, st, side, ev_fork,
                             ev_join);
}

hipError_t sorf_launch_solve_f64(int32_t D, const double* G, const double* Zty, double lambda,
                                 int32_t n_refine, double* alpha, int32_t* info, void* ws,
                                 hipStream_t st, hipStream_t side, hipEvent_t ev_fork,
                                 hipEvent_t ev_join) {
  return launch_solve<double>(D, G, Zty, lambda, n_refine, alpha, info, ws, st, side, ev_fork,
                              ev_join);
}
