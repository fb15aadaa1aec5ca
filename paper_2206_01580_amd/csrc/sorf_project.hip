// Per-element projection of the atomic representation to d = 2^n entries
// (arXiv 2206.01580, Theory section, SORF subsection): x_i = rho_i^T U_{e_i},
// where U_e holds the first d left singular vectors of element e's sampled
// representations. Every element has its own matrix, so the product is a
// grouped GEMM: the atoms are bucketed by element, and each bucket is
// multiplied by its element's d_rep x d matrix on the FP32 matrix cores.
//
// Launches:
//   count    per-element atom counts (LDS histogram per block, then one
//            integer atomic per element and block);
//   offsets  one block: bucket offsets, bucket cursors and tile offsets;
//   scatter  every atom takes a slot of its element's bucket (a block
//            reserves its atoms' ranges with one atomic per element); the
//            order inside a bucket varies between runs, but each output row
//            depends on its own input row only, so x does not;
//            (up to kProjFewAtoms atoms one kernel does all three);
//   gemm     one workgroup per 128 atoms of one bucket x 128 output columns
//            (32 where that would leave compute units idle).
//            rho rows are gathered through the bucket list into LDS as
//            [k][atom], U_e rows as [k][column], both double-buffered in
//            chunks of 16 k with the next chunk held in registers while the
//            current one is multiplied. Each wave owns 32 atoms x 128 columns
//            (4 blocks of v_mfma_f32_32x32x2f32) and writes its rows once.
#include "sorf_internal.h"

namespace sorf {

constexpr int kProjRows = 128;   // atoms per tile
constexpr int kProjCols = 128;   // output columns per tile
constexpr int kProjK = 16;       // k per LDS stage
constexpr int kProjMaxElements = 256;

typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256) void proj_count_kernel(const int32_t* __restrict__ element,
                                                         int64_t n, int32_t E,
                                                         unsigned long long* __restrict__ counts) {
  __shared__ unsigned int h[kProjMaxElements];
  for (int i = threadIdx.x; i < E; i += blockDim.x) h[i] = 0u;
  __syncthreads();
  for (int64_t a = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; a < n;
       a += int64_t(gridDim.x) * blockDim.x) {
    const int32_t e = element[a];
    if (e >= 0 && e < E) atomicAdd(&h[e], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < E; i += blockDim.x)
    if (h[i] != 0u) atomicAdd(&counts[i], static_cast<unsigned long long>(h[i]));
}

// off[e] = atoms of elements before e; cursor[e] = off[e]; tiles[e] = tiles of
// elements before e (tiles[E] = all tiles).
__global__ void proj_offsets_kernel(const unsigned long long* __restrict__ counts, int32_t E,
                                    int64_t* __restrict__ off,
                                    unsigned long long* __restrict__ cursor,
                                    int64_t* __restrict__ tiles) {
  if (threadIdx.x != 0) return;
  int64_t o = 0, t = 0;
  for (int32_t e = 0; e < E; ++e) {
    off[e] = o;
    cursor[e] = static_cast<unsigned long long>(o);
    tiles[e] = t;
    const int64_t c = int64_t(counts[e]);
    o += c;
    t += (c + kProjRows - 1) / kProjRows;
  }
  off[E] = o;
  tiles[E] = t;
}

// A block owns a contiguous run of atoms. It counts them per element in LDS,
// reserves each element's range in the bucket with one global atomic, and
// hands out the slots of that range with LDS atomics.
__global__ __launch_bounds__(256) void proj_scatter_kernel(const int32_t* __restrict__ element,
                                                           int64_t n, int32_t E,
                                                           unsigned long long* __restrict__ cursor,
                                                           int64_t* __restrict__ perm) {
  __shared__ unsigned int h[kProjMaxElements];
  __shared__ unsigned long long base[kProjMaxElements];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t a0 = int64_t(blockIdx.x) * per;
  const int64_t a1 = a0 + per < n ? a0 + per : n;
  for (int i = threadIdx.x; i < E; i += blockDim.x) h[i] = 0u;
  __syncthreads();
  for (int64_t a = a0 + threadIdx.x; a < a1; a += blockDim.x) {
    const int32_t e = element[a];
    if (e >= 0 && e < E) atomicAdd(&h[e], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < E; i += blockDim.x) {
    base[i] = h[i] != 0u ? atomicAdd(&cursor[i], static_cast<unsigned long long>(h[i])) : 0ull;
    h[i] = 0u;
  }
  __syncthreads();
  for (int64_t a = a0 + threadIdx.x; a < a1; a += blockDim.x) {
    const int32_t e = element[a];
    if (e >= 0 && e < E) perm[int64_t(base[e] + atomicAdd(&h[e], 1u))] = a;
  }
}

// The same three steps for few atoms, in one workgroup: counts, offsets and
// slots in LDS. One launch where the kernels above take four with a fill;
// above kProjFewAtoms one workgroup's walk over the atoms is the longer.
constexpr int64_t kProjFewAtoms = 4096;
__global__ __launch_bounds__(1024) void proj_bucket_kernel(const int32_t* __restrict__ element,
                                                           int64_t n, int32_t E,
                                                           int64_t* __restrict__ off,
                                                           int64_t* __restrict__ tiles,
                                                           int64_t* __restrict__ perm) {
  __shared__ unsigned int h[kProjMaxElements], base[kProjMaxElements];
  const int tid = threadIdx.x;
  if (tid < E) h[tid] = 0u;
  __syncthreads();
  for (int64_t a = tid; a < n; a += 1024) {
    const int32_t e = element[a];
    if (e >= 0 && e < E) atomicAdd(&h[e], 1u);
  }
  __syncthreads();
  if (tid == 0) {
    unsigned int o = 0, t = 0;
    for (int32_t e = 0; e < E; ++e) {
      off[e] = o;
      tiles[e] = t;
      base[e] = o;
      o += h[e];
      t += (h[e] + kProjRows - 1) / kProjRows;
    }
    off[E] = o;
    tiles[E] = t;
  }
  __syncthreads();
  for (int64_t a = tid; a < n; a += 1024) {
    const int32_t e = element[a];
    if (e >= 0 && e < E) perm[atomicAdd(&base[e], 1u)] = a;
  }
}

// COLS output columns and KST k a stage. 128 and 16: the large tile for many
// atoms, bound by the FP32 matrix cores. 32 and 64: for calls whose large tiles
// would leave compute units idle: a quarter of the products a wave, and a
// stage long enough that the next one's loads arrive meanwhile (21 atoms,
// 720 -> 128: 32 us, now 14). Every output is the same chain of products
// over k in both, so the bits do not depend on the choice.
template <bool VEC4, int COLS, int KST>
__global__ __launch_bounds__(256) void proj_gemm_kernel(
    const float* __restrict__ rho, int32_t d_rep, const float* __restrict__ U, int32_t d,
    int32_t E, const int64_t* __restrict__ off, const int64_t* __restrict__ tiles,
    const int64_t* __restrict__ perm, float* __restrict__ x) {
  constexpr int LDA = kProjRows + 4, LDB = COLS + 4, NB = COLS / 32;
  constexpr int AK = kProjRows * KST / 256;      // k of A per thread
  constexpr int BT = COLS / 8;                   // threads of a row of B
  static_assert(256 / BT == KST && AK % 4 == 0, "one pass of the workgroup per stage");
  __shared__ float sA[2][KST][LDA];
  __shared__ __attribute__((aligned(16))) float sB[2][KST][LDB];
  __shared__ int64_t sPerm[kProjRows];

  // tile -> (element, first bucket slot)
  const int64_t t = blockIdx.x;
  if (t >= tiles[E]) return;
  int32_t e = 0;
  while (t >= tiles[e + 1]) ++e;
  const int64_t r0 = off[e] + (t - tiles[e]) * kProjRows;
  const int nrows = int(off[e + 1] - r0 < kProjRows ? off[e + 1] - r0 : kProjRows);
  const int64_t c0 = int64_t(blockIdx.y) * COLS;
  const int ncols = int(d - c0 < COLS ? d - c0 : COLS);
  const float* __restrict__ Ue = U + int64_t(e) * d_rep * d;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  if (tid < kProjRows) sPerm[tid] = perm[r0 + (tid < nrows ? tid : nrows - 1)];
  __syncthreads();

  // A: thread -> atom tid / 2, AK consecutive k; B: one k, 8 columns
  const int ar = tid >> 1, ak = (tid & 1) * AK;
  const int bk = tid / BT, bc = (tid % BT) * 8;
  const float* __restrict__ arow = rho + sPerm[ar] * int64_t(d_rep);
  float pa[AK], pb[8];
  auto load = [&](int k0) {
    const int ka = k0 + ak;
    if (VEC4 && ka + AK <= d_rep) {
#pragma unroll
      for (int j = 0; j < AK; j += 4) {
        const float4 u = *reinterpret_cast<const float4*>(arow + ka + j);
        pa[j] = u.x; pa[j + 1] = u.y; pa[j + 2] = u.z; pa[j + 3] = u.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < AK; ++j) {
        const int k = ka + j;
        const float v = arow[k < d_rep ? k : d_rep - 1];
        pa[j] = k < d_rep ? v : 0.0f;
      }
    }
    const int kb = k0 + bk;
    const int64_t cb = c0 + bc;
    const int kbc = kb < d_rep ? kb : d_rep - 1;
    const float* __restrict__ brow = Ue + int64_t(kbc) * d;
    if (VEC4 && kb < d_rep && cb + 8 <= d) {
      const float4 u = *reinterpret_cast<const float4*>(brow + cb);
      const float4 w = *reinterpret_cast<const float4*>(brow + cb + 4);
      pb[0] = u.x; pb[1] = u.y; pb[2] = u.z; pb[3] = u.w;
      pb[4] = w.x; pb[5] = w.y; pb[6] = w.z; pb[7] = w.w;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int64_t c = cb + j;
        const float v = brow[c < d ? c : d - 1];
        pb[j] = (kb < d_rep && c < d) ? v : 0.0f;
      }
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < AK; ++j) sA[buf][ak + j][ar] = pa[j];
    *reinterpret_cast<float4*>(&sB[buf][bk][bc]) = make_float4(pb[0], pb[1], pb[2], pb[3]);
    *reinterpret_cast<float4*>(&sB[buf][bk][bc + 4]) = make_float4(pb[4], pb[5], pb[6], pb[7]);
  };

  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;

  const bool busy = __builtin_amdgcn_readfirstlane(wv) * 32 < nrows;   // a wave with rows
  const int n_stages = (d_rep + KST - 1) / KST;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < n_stages; ++s) {
    const int buf = s & 1;
    if (s + 1 < n_stages) load((s + 1) * KST);
    if (COLS == kProjCols || busy) {
#pragma unroll
      for (int kb = 0; kb < KST; kb += 16) {
        if (kb > 0 && s * KST + kb >= d_rep) break;
#pragma unroll
        for (int kk = kb; kk < kb + 16; kk += 2) {
          const int k = kk + (lane >> 5);
          const float a = sA[buf][k][wv * 32 + (lane & 31)];
          float bv[NB];
#pragma unroll
          for (int b = 0; b < NB; ++b) bv[b] = sB[buf][k][b * 32 + (lane & 31)];
#pragma unroll
          for (int b = 0; b < NB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, bv[b], acc[b], 0, 0, 0);
        }
      }
    }
    if (s + 1 < n_stages) store(buf ^ 1);
    __syncthreads();
  }

#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = wv * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      const int col = b * 32 + (lane & 31);
      if (row < nrows && col < ncols) x[sPerm[row] * int64_t(d) + c0 + col] = acc[b][r];
    }
}

}  // namespace sorf

using namespace sorf;

size_t sorf_project_ws_bytes(int64_t n_atoms, int32_t n_elements) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t E = size_t(n_elements);
  return al(8 * E) + al(8 * (E + 1)) + al(8 * E) + al(8 * (E + 1)) + al(8 * size_t(n_atoms));
}

hipError_t sorf_launch_project(int64_t n_atoms, int32_t d_rep, const float* rho,
                               const int32_t* element, int32_t E, const float* U, int32_t d,
                               float* x, void* ws, hipStream_t st) {
  if (n_atoms == 0) return hipSuccess;
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  char* p = static_cast<char*>(ws);
  auto* counts = reinterpret_cast<unsigned long long*>(p);
  p += al(8 * size_t(E));
  auto* off = reinterpret_cast<int64_t*>(p);
  p += al(8 * size_t(E + 1));
  auto* cursor = reinterpret_cast<unsigned long long*>(p);
  p += al(8 * size_t(E));
  auto* tiles = reinterpret_cast<int64_t*>(p);
  p += al(8 * size_t(E + 1));
  auto* perm = reinterpret_cast<int64_t*>(p);

  if (n_atoms <= kProjFewAtoms) {
    hipLaunchKernelGGL(proj_bucket_kernel, dim3(1), dim3(1024), 0, st, element, n_atoms, E, off,
                       tiles, perm);
  } else {
    // counts start at zero: a fill kernel, not a memset, so the call can be captured
    hipError_t err = sorf_launch_fill(reinterpret_cast<float*>(counts), 2 * int64_t(E), 0.0f, st);
    if (err != hipSuccess) return err;
    int64_t blocks = (n_atoms + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(proj_count_kernel, dim3(unsigned(blocks)), dim3(256), 0, st, element,
                       n_atoms, E, counts);
    hipLaunchKernelGGL(proj_offsets_kernel, dim3(1), dim3(64), 0, st, counts, E, off, cursor,
                       tiles);
    hipLaunchKernelGGL(proj_scatter_kernel, dim3(unsigned(blocks)), dim3(256), 0, st, element,
                       n_atoms, E, cursor, perm);
  }
  // at most ceil(A / 128) + E tiles; blocks past the real count exit
  const int64_t max_tiles = (n_atoms + kProjRows - 1) / kProjRows + E;
  const bool vec4 = (d_rep % 4 == 0) && (d % 4 == 0) &&
                    (reinterpret_cast<uintptr_t>(rho) & 15u) == 0 &&
                    (reinterpret_cast<uintptr_t>(U) & 15u) == 0;
  const auto go = [&](auto kernel, int cols) {
    const dim3 grid(unsigned(max_tiles), unsigned((d + cols - 1) / cols));
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, rho, d_rep, U, d, E, off, tiles, perm, x);
  };
  // The small tiles while two rounds of them (one fills a compute unit's LDS) cover the
  // call: a round takes 35 us at d_rep = 720, one round of large tiles 75. d = 128: 15,700
  // atoms 69 us against 76, 20,000 (three rounds) 98 against 77; d = 64: 32,000 atoms 71
  // against 100.
  if (max_tiles * ((d + 31) / 32) <= 512)
    vec4 ? go(proj_gemm_kernel<true, 32, 64>, 32) : go(proj_gemm_kernel<false, 32, 64>, 32);
  else
    vec4 ? go(proj_gemm_kernel<true, kProjCols, kProjK>, kProjCols)
         : go(proj_gemm_kernel<false, kProjCols, kProjK>, kProjCols);
  return hipGetLastError();
}
