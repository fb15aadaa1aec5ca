// FCHL19 atomic representation (arXiv 2206.01580, Theory section,
// Representation subsection; parameters from the Computational Details
// table): for every atom i,
//   rho_i = [G2_X for every element X] ++ [G3_XY for every element pair X <= Y],
//   G2_X[k]     = sum_{j in X} f_cut(r_ij) r_ij^-N2 LN(R_k; mu(r_ij), sigma(r_ij)),
//                 LN the log-normal density, mu = ln(r / sqrt(1 + eta2/r^2)),
//                 sigma^2 = ln(1 + eta2/r^2), R_k = r_cut (k + 1) / n2;
//   G3_XY[k][t] = sum over unordered neighbour pairs {j, k'} of elements {X, Y} of
//                 xi3 f_cut(r_ij) f_cut(r_jk') f_cut(r_ik') sqrt(eta3/pi)
//                 exp(-eta3 ((r_ij + r_ik')/2 - R_k)^2) A_t(theta),
//                 xi3 = c3 (1 + 3 cos_i cos_j cos_k') / (r_ij r_jk' r_ik')^N3 (Axilrod-Teller-Muto),
//                 A_cos = 2 e^(-zeta^2/2) cos(theta), A_sin = 2 e^(-zeta^2/2) sin(theta),
//                 theta the angle at i, R_k = r_cut k / (n3 - 1); f_cut(r) = (cos(pi r/r_cut) + 1)/2
//                 below r_cut and 0 beyond.
//
// Atoms of molecules of up to 64 atoms take one wave each (see
// fchl19_forward_small_kernel). Larger molecules: one workgroup per atom, of 16
// waves, or of 8 from 257 atoms in the batch on (fchl_few_atoms). The atom's
// neighbours (same molecule, closer than r_cut) are gathered into LDS grouped by
// element, in atom order inside each group (ballot compaction, no atomics), with their per-neighbour
// two-body factors. Two-body bins: one thread per (element, bin) sums its
// element's neighbours in order. Three-body: the unordered pairs are numbered
// by element pair (X <= Y), then by position; chunks of pairs get their
// radial-independent weight (xi3, cutoffs, angle) computed by all threads
// into LDS, and groups of one thread per radial bin sum equal parts of
// the chunk in order. Every entry of rho is therefore summed in a fixed order.
#include <cmath>

#include "sorf_internal.h"

namespace sorf {

constexpr int kFchlMaxNb = 512;        // neighbours of one atom held in LDS
constexpr int kFchlPairChunk = 2048;   // three-body pairs per LDS chunk
// Least pairs of a group's part of a chunk. The group in whose part an element pair ends
// adds up the earlier ones', one after the other: with two radial bins (512 groups) this
// took most of the time, 178 us for 245 atoms, now 72.
constexpr int kFchlPartPairs = 8;
constexpr int kFchlMaxElements = 16;
constexpr int kFchlSmallMol = 64;       // molecules up to this size take the wave-per-atom kernel

struct FchlParams {
  int32_t n2, n3;
  float eta2, eta3, N2, N3, c3, zeta, rcut;
};

// The argument of the cutoff's cosine, pi r / r_cut, lies in [0, pi) below
// r_cut, so the hardware sine and cosine (argument in revolutions, here in
// [0, 1/2)) serve without range reduction; f_cut is exactly 0 at and beyond r_cut.
__device__ __forceinline__ float fchl_fcut(float r, float rc) {
  return r < rc ? 0.5f * (__builtin_amdgcn_cosf(r * (0.5f / rc)) + 1.0f) : 0.0f;
}
// d f_cut / dr
__device__ __forceinline__ float fchl_dfcut(float r, float rc) {
  return r < rc ? -0.5f * (3.14159265358979f / rc) * __builtin_amdgcn_sinf(r * (0.5f / rc)) : 0.0f;
}

// Hardware exp2, log2 and reciprocal (about 1 ulp each) for the radial-bin
// loops, where the correctly rounded library sequences cost several times
// as many instructions; arguments there are at most a few tens in magnitude,
// so the results keep a relative accuracy of about 1e-6.
__device__ __forceinline__ float fchl_exp(float x) {
  return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
}
__device__ __forceinline__ float fchl_ln(float x) {
  return __builtin_amdgcn_logf(x) * 0.693147180559945309f;
}
__device__ __forceinline__ float fchl_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// element pair (a <= b) -> position in the lexicographic list of pairs
__device__ __forceinline__ int fchl_pair(int a, int b, int E) { return a * E - a * (a - 1) / 2 + (b - a); }

// loc / c for 0 <= loc < 2^22 and c >= 1: the FP32 quotient is off by one at most.
__device__ __forceinline__ int fchl_div(int loc, int c) {
  int u = int(float(loc) * fchl_rcp(float(c)));
  u -= u * c > loc ? 1 : 0;
  u += (u + 1) * c <= loc ? 1 : 0;
  return u;
}
// Row u of the pairs (u, v), u < v < n, numbered row by row; row u starts at u (2 n - u - 1) / 2.
// (n at most 512, so the discriminant is exact in FP32)
__device__ __forceinline__ int fchl_pair_row(int loc, int n) {
  const float c2n = 2.0f * float(n) - 1.0f;
  int u = int((c2n - __builtin_amdgcn_sqrtf(c2n * c2n - 8.0f * float(loc))) * 0.5f);
  u = u < 0 ? 0 : (u > n - 2 ? n - 2 : u);
  while (u > 0 && u * (2 * n - u - 1) / 2 > loc) --u;
  while ((u + 1) * (2 * n - u - 2) / 2 <= loc) ++u;
  return u;
}

constexpr int kFchlThreads = 1024;   // workgroup of the kernels for large molecules

// The neighbours of atom i (atoms a0 .. a1 - 1 closer than r_cut), grouped by
// element, atom order inside a group: store(slot, j, dx, dy, dz, r) for every
// one of the first kFchlMaxNb, grp[X] the first slot of element X, grp[E] the
// number of all. A wave takes a contiguous run of atoms, counts its
// neighbours per element with ballots (lane X keeps element X's count), one
// wave turns the counts into first slots, and each wave hands out its own:
// two barriers for any molecule, where a pass per element and 1024 atoms had
// one each and formed the neighbours' factors anew in each (1260 atoms, 16
// waves: the forward 173 us, now 133, the backward 167, now 132).
template <int NT>
struct FchlGather {
  int32_t first[kFchlMaxElements][NT / 64];
  int32_t grp[kFchlMaxElements + 1];
};
template <int NT, typename Store>
__device__ __forceinline__ int fchl_gather(int64_t i, int64_t a0, int64_t a1,
                                           const float* __restrict__ R,
                                           const int32_t* __restrict__ element, int32_t E,
                                           float rc, FchlGather<NT>& sh, Store store) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float xi = R[3 * i], yi = R[3 * i + 1], zi = R[3 * i + 2];
  const int64_t pieces = (a1 - a0 + 64 * NW - 1) / (64 * NW);   // of 64 atoms, per wave
  const int64_t w0 = a0 + wv * pieces * 64;
  float dx = 0.f, dy = 0.f, dz = 0.f, r = 0.f;
  int e = -1;   // this lane's element if it holds a neighbour
  const auto piece = [&](int64_t j) {
    e = -1;
    if (j < a1 && j != i) {
      dx = R[3 * j] - xi;
      dy = R[3 * j + 1] - yi;
      dz = R[3 * j + 2] - zi;
      r = sqrtf(dx * dx + dy * dy + dz * dz);
      if (r < rc) e = element[j];
    }
  };
  int count = 0;
  for (int64_t p = 0; p < pieces; ++p) {
    piece(w0 + 64 * p + lane);
    for (int X = 0; X < E; ++X) {
      const int n = __popcll(__ballot(e == X));
      count += lane == X ? n : 0;
    }
  }
  if (lane < E) sh.first[lane][wv] = count;
  __syncthreads();
  if (wv == 0) {   // exclusive sums over (element, wave), four waves' counts a lane
    int v[NW / 4], sum = 0;
    int32_t* const c = &sh.first[lane / 4][(lane % 4) * (NW / 4)];
#pragma unroll
    for (int t = 0; t < NW / 4; ++t) {
      v[t] = lane / 4 < E ? c[t] : 0;
      sum += v[t];
    }
    int before = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(before, o);
      before += lane >= o ? up : 0;
    }
    if (lane == 63) sh.grp[E] = before;
    before -= sum;
    if (lane / 4 < E) {
      if (lane % 4 == 0) sh.grp[lane / 4] = before;
#pragma unroll
      for (int t = 0; t < NW / 4; ++t) {
        c[t] = before;
        before += v[t];
      }
    }
  }
  __syncthreads();
  int next = lane < E ? sh.first[lane][wv] : 0;   // lane X: element X's next slot of this wave
  for (int64_t p = 0; p < pieces; ++p) {
    if (pieces > 1) piece(w0 + 64 * p + lane);
    int slot = kFchlMaxNb;
    for (int X = 0; X < E; ++X) {
      const uint64_t mask = __ballot(e == X);
      const int s0 = __shfl(next, X);
      if (e == X) slot = s0 + __popcll(mask & ((uint64_t(1) << lane) - 1));
      next += lane == X ? __popcll(mask) : 0;
    }
    if (slot < kFchlMaxNb) store(slot, w0 + 64 * p + lane, dx, dy, dz, r);
  }
  return sh.grp[E];
}

// Pairs of neighbours numbered by element pair X <= Y, then by position: seg[P] the
// first of element pair P, seg[NP] their number, xy[P] = X | Y << 8. One thread per
// element pair (one thread for all took a third of the time of an atom with few
// neighbours and 16 elements).
template <int NT>
__device__ __forceinline__ void fchl_segments(const int32_t* grp, int E, int32_t* seg, int32_t* xy) {
  const int NP = E * (E + 1) / 2, n = grp[E];
  for (int P = threadIdx.x; P < NP; P += NT) {
    int X = 0;
    while (fchl_pair(X, X, E) + (E - X) <= P) ++X;
    const int Y = X + (P - fchl_pair(X, X, E));
    // pairs whose first neighbour comes before X's, then those of X before Y's
    const int gX = grp[X], cx = grp[X + 1] - gX;
    int32_t o = gX * (2 * n - gX - 1) / 2;
    if (Y > X) o += cx * (cx - 1) / 2 + cx * (grp[Y] - grp[X + 1]);
    seg[P] = o;
    xy[P] = X | (Y << 8);
  }
  if (threadIdx.x == 0) seg[NP] = n * (n - 1) / 2;
}

// Atom i of molecule m (atoms a0 .. a1 - 1), a workgroup of NT threads. The sums
// are those of kFchlThreads threads with either NT, so the bits are the same.
//
// Bound by vector issue: the pair weights (about 150 instructions a pair) and
// the radial bins (an exponential and about ten instructions a pair and bin).
// What depends on one neighbour alone (1 / r, r^-N3 f_cut) is formed
// once per neighbour. The bins of a chunk are split over groups of one thread
// per radial bin, each with an equal part of the chunk's pairs in order; one
// thread per (element pair, bin) left all but the largest element pair's
// threads idle (182 us for the 245 atoms of a cluster, now 37).
template <int NT>
__device__ __forceinline__ void fchl19_forward_atom(
    int64_t i, int64_t a0, int64_t a1, const float* __restrict__ R,
    const int32_t* __restrict__ element, int32_t E, const FchlParams& p, int64_t size,
    float* __restrict__ rho) {
  constexpr int VT = kFchlThreads;
  __shared__ float nx[kFchlMaxNb], ny[kFchlMaxNb], nz[kFchlMaxNb], nr[kFchlMaxNb];
  __shared__ float ni[kFchlMaxNb], nw[kFchlMaxNb], c2[kFchlMaxNb], mu2[kFchlMaxNb], inv2s2[kFchlMaxNb];
  __shared__ FchlGather<NT> gathered;
  __shared__ int32_t seg[kFchlMaxElements * (kFchlMaxElements + 1) / 2 + 1];
  __shared__ int32_t pair_xy[kFchlMaxElements * (kFchlMaxElements + 1) / 2];
  __shared__ float4 pw[kFchlPairChunk];             // w cos, w sin, mean distance
  __shared__ float2 tail[VT], head[NT < VT ? VT : 1];
  __shared__ int32_t ends[NT < VT ? VT / 2 : 1];    // n3 >= 2

  const int tid = threadIdx.x;
  const float rc = p.rcut;
  float* __restrict__ out = rho + i * size;
  const int32_t* const grp = gathered.grp;          // neighbour offsets per element
  const int total = fchl_gather<NT>(
      i, a0, a1, R, element, E, rc, gathered,
      [&](int slot, int64_t, float dx, float dy, float dz, float r) {
        // f_cut as sin^2(pi (r_cut - r) / (2 r_cut)), without the cancellation of
        // (cos + 1) / 2 near the cutoff
        const float sc = sinf(1.57079632679490f * ((rc - r) / rc));
        const float fc = sc * sc;
        nx[slot] = dx;
        ny[slot] = dy;
        nz[slot] = dz;
        nr[slot] = r;
        ni[slot] = 1.0f / r;
        nw[slot] = powf(r, -p.N3) * fc;
        // two-body factors: f_cut r^-N2 / (sigma sqrt(2 pi)), mu, 1 / (2 sigma^2)
        const float q = 1.0f + p.eta2 / (r * r);
        const float s2 = logf(q);
        c2[slot] = fc * powf(r, -p.N2) / (sqrtf(s2) * 2.50662827463100f);
        mu2[slot] = logf(r / sqrtf(q));
        inv2s2[slot] = 0.5f / s2;
      });
  if (total > kFchlMaxNb) {   // more neighbours than the LDS list holds: mark the row, do not guess
    for (int64_t t = tid; t < size; t += NT) out[t] = __builtin_nanf("");
    return;
  }
  __syncthreads();

  // three-body: pair numbering by element pair X <= Y
  const int NP = E * (E + 1) / 2;
  fchl_segments<NT>(grp, E, seg, pair_xy);

  // two-body bins
  for (int t = tid; t < E * p.n2; t += NT) {
    const int X = t / p.n2, k = t % p.n2;
    const float Rk = rc * float(k + 1) / float(p.n2);
    const float lnR = logf(Rk);
    float acc = 0.0f;
    for (int s = grp[X]; s < grp[X + 1]; ++s) {
      const float d = lnR - mu2[s];
      acc += c2[s] * fchl_exp(-d * d * inv2s2[s]);
    }
    out[t] = acc / Rk;
  }
  __syncthreads();
  const int32_t n_pairs = seg[NP];
  const float angw = 2.0f * expf(-0.5f * p.zeta * p.zeta) * sqrtf(p.eta3 / 3.14159265358979f);
  const float c3w = p.c3 * angw;
  float* __restrict__ out3 = out + int64_t(E) * p.n2;
  // element pairs without pairs
  for (int t = tid; t < NP * p.n3; t += NT) {
    const int P = t / p.n3;
    if (seg[P] == seg[P + 1]) {
      out3[2 * t] = 0.0f;
      out3[2 * t + 1] = 0.0f;
    }
  }
  // G groups of n3 threads, thread kl of a group on radial bin kl; group g
  // walks the g-th of G equal parts of a chunk, of kFchlPartPairs pairs at least. An
  // element pair whose pairs fall in several parts is finished by the group where it
  // ends, which adds the earlier groups' partial sums in group order. With more radial
  // bins than threads the threads of one group loop over them. With fewer than VT
  // threads (n3 <= NT then) each group of threads takes every step-th group.
  const int most = p.n3 <= VT ? VT / p.n3 : 1;
  const int step = NT < VT ? NT / p.n3 : most;
  const int g0 = p.n3 <= NT ? tid / p.n3 : 0;
  const int kl = p.n3 <= NT ? tid % p.n3 : tid;
  const float keta = -p.eta3 * 1.44269504088896341f;
  int P = 0, Q0 = 0;   // non-decreasing over the chunks
  for (int32_t q0 = 0; q0 < n_pairs; q0 += kFchlPairChunk) {
    const int32_t q1 = q0 + kFchlPairChunk < n_pairs ? q0 + kFchlPairChunk : n_pairs;
    for (int32_t q = q0 + tid; q < q1; q += NT) {
      // pair q -> element pair P (row X, column Y) -> neighbours (a, b)
      while (q >= seg[P + 1]) ++P;
      const int X = pair_xy[P] & 255, Y = pair_xy[P] >> 8;
      const int32_t loc = q - seg[P];
      int a, b;
      if (X != Y) {
        const int cy = grp[Y + 1] - grp[Y];
        const int u = fchl_div(loc, cy);
        a = grp[X] + u;
        b = grp[Y] + loc - u * cy;
      } else {
        const int cx = grp[X + 1] - grp[X];
        const int u = fchl_pair_row(loc, cx);
        a = grp[X] + u;
        b = grp[X] + u + 1 + (loc - u * (2 * cx - u - 1) / 2);
      }
      const float rij = nr[a], rik = nr[b];
      const float ax = nx[a], ay = ny[a], az = nz[a], bx = nx[b], by = ny[b], bz = nz[b];
      const float jx = bx - ax, jy = by - ay, jz = bz - az;
      const float rjk = sqrtf(jx * jx + jy * jy + jz * jz);
      float ijk = fchl_rcp(rjk);
      ijk = __builtin_fmaf(__builtin_fmaf(-rjk, ijk, 1.0f), ijk, ijk);
      const float iij = ni[a], iik = ni[b];
      const float cos_i = (ax * bx + ay * by + az * bz) * (iij * iik);
      const float cos_j = -(ax * jx + ay * jy + az * jz) * (iij * ijk);
      const float cos_k = (bx * jx + by * jy + bz * jz) * (iik * ijk);
      const float sin_i = sqrtf(fmaxf(0.0f, 1.0f - cos_i * cos_i));
      const float w = c3w * (1.0f + 3.0f * cos_i * cos_j * cos_k) * (nw[a] * nw[b]) *
                      (__builtin_amdgcn_exp2f(-p.N3 * __builtin_amdgcn_logf(rjk)) *
                       fchl_fcut(rjk, rc));
      pw[q - q0] = make_float4(w * cos_i, w * sin_i, 0.5f * (rij + rik), 0.0f);
    }
    __syncthreads();
    const int32_t L = q1 - q0;
    const int G = min(most, (L + kFchlPartPairs - 1) / kFchlPartPairs);
    // Radial bin k of group g's part: adds up the element pairs that begin and end in it,
    // returns the one (or -1) that only ends in it with its sums (pc, ps), and leaves
    // the sums of the one that is open at the part's end in tail.
    const auto part = [&](int g, int k, int& Q0, float& pc, float& ps) {
      int pend = -1;
      const float Rk = rc * float(k) / float(p.n3 - 1);
      const int32_t lo = q0 + L * g / G, hi = q0 + L * (g + 1) / G;
      while (Q0 < NP && seg[Q0 + 1] <= lo) ++Q0;
      int Q = Q0;
      bool started = Q < NP && (seg[Q] > q0 ? seg[Q] : q0) >= lo;
      float c = 0.f, sn = 0.f;
      for (int32_t q = lo; q < hi;) {
        const int32_t segend = seg[Q + 1] < q1 ? seg[Q + 1] : q1;
        const int32_t stop = segend < hi ? segend : hi;
#pragma unroll 4
        for (; q < stop; ++q) {
          const float4 w = pw[q - q0];
          const float d = w.z - Rk;
          const float gk = __builtin_amdgcn_exp2f(keta * (d * d));
          c = __builtin_fmaf(w.x, gk, c);
          sn = __builtin_fmaf(w.y, gk, sn);
        }
        if (q == segend) {              // element pair Q ends in this part
          if (started) {
            float* o = out3 + 2 * (int64_t(Q) * p.n3 + k);
            const bool first = seg[Q] >= q0;
            o[0] = first ? c : o[0] + c;
            o[1] = first ? sn : o[1] + sn;
          } else {
            pend = Q;
            pc = c;
            ps = sn;
          }
          c = 0.f;
          sn = 0.f;
          ++Q;
          while (Q < NP && seg[Q + 1] <= q) ++Q;
          started = true;
        }
      }
      tail[g * p.n3 + (p.n3 <= VT ? k : tid)] = make_float2(c, sn);   // 0 if none is open
      return pend;
    };
    // Element pair Q, which ends in group g's part with the sums (pc, ps) and began earlier.
    const auto finish = [&](int g, int k, int Q, float pc, float ps) {
      const int32_t st = seg[Q] > q0 ? seg[Q] : q0;
      int gs = g - 1;                   // the group in whose part the element pair starts
      while (gs > 0 && q0 + L * gs / G > st) --gs;
      float sc = 0.f, ss = 0.f;
      for (int gg = gs; gg < g; ++gg) {
        sc += tail[gg * p.n3 + k].x;
        ss += tail[gg * p.n3 + k].y;
      }
      float* o = out3 + 2 * (int64_t(Q) * p.n3 + k);
      const bool first = seg[Q] >= q0;
      o[0] = first ? sc + pc : o[0] + (sc + pc);
      o[1] = first ? ss + ps : o[1] + (ss + ps);
    };
    if constexpr (NT == VT) {
      int pend = -1;
      float pc = 0.f, ps = 0.f;
      for (int k = kl; k < p.n3 && g0 < G; k += NT) pend = part(g0, k, Q0, pc, ps);
      __syncthreads();
      if (pend >= 0) finish(g0, kl, pend, pc, ps);
    } else {
      int Qg = Q0;
      for (int g = g0; g < G && g0 < step; g += step) {
        float pc = 0.f, ps = 0.f;
        const int pend = part(g, kl, Qg, pc, ps);
        head[g * p.n3 + kl] = make_float2(pc, ps);
        if (kl == 0) ends[g] = pend;
        if (g == g0) Q0 = Qg;
      }
      __syncthreads();
      for (int g = g0; g < G && g0 < step; g += step)
        if (ends[g] >= 0) {
          const float2 h = head[g * p.n3 + kl];
          finish(g, kl, ends[g], h.x, h.y);
        }
    }
    __syncthreads();   // weights and tails are reused, and the next chunk adds to these entries
  }
}

// Atoms of larger molecules: a persistent grid in which every workgroup reads
// the molecule sizes NT at a time (coalesced), collects the molecules above
// kFchlSmallMol atoms with ballots, and takes those of their atoms whose index in
// the batch is its own modulo the grid, so that the atoms of one large molecule and
// of several spread evenly (from (m + j) mod grid on for atom j of molecule m, a
// hundred molecules of 65 atoms shared a quarter of the workgroups). What the walk
// over the molecules needs is in LDS.
template <int NT>
struct FchlDeal {
  int64_t a0[NT], n[NT];   // first atom, atoms
  int32_t shift[NT];       // first atom mod grid
  int32_t per_wave[2][NT / 64];   // of this group of molecules and the next
};
template <int NT, typename Atom>
__device__ __forceinline__ void fchl_deal(const int64_t* __restrict__ mol_ptr, int64_t n_mols,
                                          int small, FchlDeal<NT>& sh, Atom atom) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t G = int32_t(gridDim.x), b = int32_t(blockIdx.x);
  int64_t lo = 0, hi = 0;
  if (tid < n_mols) {
    lo = mol_ptr[tid];
    hi = mol_ptr[tid + 1];
  }
  int buf = 0;
  for (int64_t m0 = 0; m0 < n_mols; m0 += NT, buf ^= 1) {
    const int64_t m = m0 + tid, a0 = lo, n = hi - lo;
    const bool large = m < n_mols && n > small;
    // next group's sizes in flight while this group is processed
    if (m + NT < n_mols) {
      lo = mol_ptr[m + NT];
      hi = mol_ptr[m + NT + 1];
    }
    const uint64_t mask = __ballot(large);
    if (lane == 0) sh.per_wave[buf][wv] = __popcll(mask);
    __syncthreads();
    int off = 0, nbig = 0;
    for (int w = 0; w < NW; ++w) {
      off += w < wv ? sh.per_wave[buf][w] : 0;
      nbig += sh.per_wave[buf][w];
    }
    if (nbig == 0) continue;   // one barrier a group of small molecules
    if (large) {
      const int t = off + __popcll(mask & ((uint64_t(1) << lane) - 1));
      sh.a0[t] = a0;
      sh.n[t] = n;
      sh.shift[t] = int32_t(uint64_t(a0) % uint32_t(G));
    }
    __syncthreads();
    for (int t = 0; t < nbig; ++t) {
      const int32_t j0 = b - sh.shift[t];
      const int64_t n_t = sh.n[t];
      for (int64_t j = j0 < 0 ? j0 + G : j0; j < n_t; j += G)
        atom(sh.a0[t] + j, sh.a0[t], sh.a0[t] + n_t);
    }
    __syncthreads();   // the list is rewritten by the next group
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void fchl19_forward_kernel(
    const float* __restrict__ R, const int32_t* __restrict__ element,
    const int64_t* __restrict__ mol_ptr, int64_t n_mols, int32_t E, FchlParams p,
    int64_t size, float* __restrict__ rho) {
  __shared__ FchlDeal<NT> deal;
  fchl_deal<NT>(mol_ptr, n_mols, kFchlSmallMol, deal, [&](int64_t i, int64_t a0, int64_t a1) {
    fchl19_forward_atom<NT>(i, a0, a1, R, element, E, p, size, rho);
    __syncthreads();   // the next atom reuses the LDS
  });
}

// Atoms of molecules of at most kFchlSmallMol atoms: one wave per atom, four
// atoms per workgroup, no workgroup barriers. The wave's lanes take the
// molecule's atoms, gather the neighbours by element with ballots into the
// wave's LDS, form the two-body bins (lanes over bins), then the three-body
// pair weights in chunks (lanes over pairs) and the three-body bins: lane
// groups of one lane per radial bin split each chunk's pairs into equal
// parts, so that no lane walks a whole large element pair (H-C, say) while
// the others idle. Every entry is summed in a fixed order (pairs in the
// workgroup-per-atom kernel's numbering, parts in group order, chunks in
// order), so results are deterministic.
//
// Bound by vector issue (2700 instructions an atom of a QM9-sized molecule)
// and by the waves in flight: 360,000 atoms 1.81 ms, now 1.41. Seven waves a
// SIMD (registers and LDS held to that; 1.50 with what the compiler chose);
// what depends on one neighbour alone formed once for all lanes, not in each
// element's turn; integer divisions by FP32 reciprocals; the molecule
// searched by the whole wave.
constexpr int kFchlWavePairs = 192;   // a chunk; more LDS would cost waves in flight

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The molecule of atom i (the last m < n_mols with mol_ptr[m] <= i), searched
// by a whole wave with 64 probes a round: three dependent loads for 20000
// molecules, where a binary search's fifteen were a third of the small kernel's time.
__device__ __forceinline__ int64_t wave_molecule_of(const int64_t* __restrict__ mol_ptr,
                                                    int64_t n_mols, int64_t i, int lane) {
  int64_t lo = 0, len = n_mols;   // the answer lies in [lo, lo + len)
  while (len > 1) {
    const int64_t step = (len + 63) / 64;
    const int64_t probe = lo + lane * step;
    const bool below = lane * step < len && mol_ptr[probe] <= i;
    const int n = __popcll(__ballot(below));   // at least one: mol_ptr[lo] <= i
    lo += (n > 0 ? n - 1 : 0) * step;
    len = step < n_mols - lo ? step : n_mols - lo;
  }
  return lo;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7, 7))) void fchl19_forward_small_kernel(
    const float* __restrict__ R, const int32_t* __restrict__ element,
    const int64_t* __restrict__ mol_ptr, int64_t atom0, int64_t n_atoms, int64_t n_mols,
    int32_t E, FchlParams p, int64_t size, float* __restrict__ rho) {
  __shared__ float nx[4][kFchlSmallMol], ny[4][kFchlSmallMol], nz[4][kFchlSmallMol];
  __shared__ float nr[4][kFchlSmallMol], ni[4][kFchlSmallMol], nw[4][kFchlSmallMol];
  __shared__ float c2[4][kFchlSmallMol], mu2[4][kFchlSmallMol], inv2s2[4][kFchlSmallMol];
  __shared__ int32_t grp[4][kFchlMaxElements + 1];
  __shared__ int32_t seg[4][kFchlMaxElements * (kFchlMaxElements + 1) / 2 + 1];
  __shared__ float2 pw[4][kFchlWavePairs];          // w cos, w sin
  __shared__ float pmid[4][kFchlWavePairs];
  __shared__ float tail[4][64][2];
  // X | Y << 8 of an element pair, the same for every wave (each stores all of it)
  __shared__ uint16_t pair_xy[kFchlMaxElements * (kFchlMaxElements + 1) / 2];

  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t i = atom0 + int64_t(blockIdx.x) * 4 + wv;
  if (i >= n_atoms) return;                   // whole waves leave
  const int64_t m = wave_molecule_of(mol_ptr, n_mols, i, lane);
  const int64_t a0 = mol_ptr[m];
  const int N = int(mol_ptr[m + 1] - a0);
  if (N > kFchlSmallMol) return;              // fchl19_forward_kernel takes this atom
  const float rc = p.rcut;
  float* __restrict__ out = rho + i * size;

  // neighbours by element, atom order inside a group (lane = candidate atom)
  const int64_t j = a0 + lane;
  float dx = 0.f, dy = 0.f, dz = 0.f, r = 0.f;
  bool in = false;
  int ej = -1;
  if (lane < N && j != i) {
    dx = R[3 * j] - R[3 * i];
    dy = R[3 * j + 1] - R[3 * i + 1];
    dz = R[3 * j + 2] - R[3 * i + 2];
    r = sqrtf(dx * dx + dy * dy + dz * dz);
    in = r < rc;
    ej = element[j];
  }
  // what depends on one neighbour alone: 1 / r, r^-N3 f_cut, and the two-body
  // factors f_cut r^-N2 / (sigma sqrt(2 pi)), mu, 1 / (2 sigma^2)
  float inv = 0.f, w3 = 0.f, fc2 = 0.f, fmu = 0.f, fi = 0.f;
  if (in) {
    const float fc = fchl_fcut(r, rc);
    const float q = 1.0f + p.eta2 / (r * r);
    const float s2 = logf(q);
    inv = 1.0f / r;
    w3 = powf(r, -p.N3) * fc;
    fc2 = fc * powf(r, -p.N2) / (sqrtf(s2) * 2.50662827463100f);
    fmu = logf(r / sqrtf(q));
    fi = 0.5f / s2;
  }
  int n = 0;
  for (int X = 0; X < E; ++X) {
    if (lane == 0) grp[wv][X] = n;
    const bool f = in && ej == X;
    const uint64_t mask = __ballot(f);
    if (f) {
      const int sl = n + __popcll(mask & ((uint64_t(1) << lane) - 1));
      nx[wv][sl] = dx;
      ny[wv][sl] = dy;
      nz[wv][sl] = dz;
      nr[wv][sl] = r;
      ni[wv][sl] = inv;
      nw[wv][sl] = w3;
      c2[wv][sl] = fc2;
      mu2[wv][sl] = fmu;
      inv2s2[wv][sl] = fi;
    }
    n += __popcll(mask);
  }
  if (lane == 0) grp[wv][E] = n;
  wave_sync_lds();

  // two-body bins
  for (int t = lane; t < E * p.n2; t += 64) {
    const int X = fchl_div(t, p.n2), k = t - X * p.n2;
    const float Rk = rc * float(k + 1) / float(p.n2);
    const float lnR = logf(Rk);
    float acc = 0.0f;
    for (int sl = grp[wv][X]; sl < grp[wv][X + 1]; ++sl) {
      const float d = lnR - mu2[wv][sl];
      acc += c2[wv][sl] * fchl_exp(-d * d * inv2s2[wv][sl]);
    }
    out[t] = acc / Rk;
  }

  // three-body: pairs numbered by element pair, then by position (the
  // workgroup-per-atom kernel's numbering)
  const int NP = E * (E + 1) / 2;
  for (int P = lane; P < NP; P += 64) {
    int X = 0;
    while (fchl_pair(X, X, E) + (E - X) <= P) ++X;
    const int Y = X + (P - fchl_pair(X, X, E));
    // pairs whose first neighbour comes before X's, then those of X before Y's
    const int gX = grp[wv][X], cx = grp[wv][X + 1] - gX;
    int32_t o = gX * (2 * n - gX - 1) / 2;
    if (Y > X) o += cx * (cx - 1) / 2 + cx * (grp[wv][Y] - grp[wv][X + 1]);
    seg[wv][P] = o;
    pair_xy[P] = uint16_t(X | (Y << 8));
  }
  if (lane == 0) seg[wv][NP] = n * (n - 1) / 2;
  wave_sync_lds();
  const int32_t n_pairs = seg[wv][NP];
  const float angw = 2.0f * expf(-0.5f * p.zeta * p.zeta) * sqrtf(p.eta3 / 3.14159265358979f);
  const float c3w = p.c3 * angw, keta = -p.eta3 * 1.44269504088896341f;
  // Bins: G groups of n3 lanes, one lane per radial bin; group g walks the
  // g-th of G equal parts of the chunk's pairs in order. An element pair
  // whose pairs fall in several parts is finished by the group where it ends,
  // which adds the partial sums of the earlier groups in group order. With
  // more than 64 radial bins one group's lanes loop over them. At most 12 groups (16
  // pairs of a full chunk each): with 32 of two radial bins the sums over groups took
  // longer than the pairs (256 molecules of 64 atoms 219 us, now 181).
  const int G = p.n3 <= 64 ? min(64 / p.n3, 12) : 1;
  const int g = p.n3 <= 64 ? lane / p.n3 : 0;
  const int kl = p.n3 <= 64 ? lane % p.n3 : lane;
  float* __restrict__ out3 = out + int64_t(E) * p.n2;
  int P = 0;   // decode state: non-decreasing in q, kept across iterations
  for (int32_t q0 = 0; q0 < n_pairs || q0 == 0; q0 += kFchlWavePairs) {
    const int32_t q1 = q0 + kFchlWavePairs < n_pairs ? q0 + kFchlWavePairs : n_pairs;
    for (int32_t q = q0 + lane; q < q1; q += 64) {
      while (q >= seg[wv][P + 1]) ++P;
      const int X = pair_xy[P] & 255, Y = pair_xy[P] >> 8;
      const int32_t loc = q - seg[wv][P];
      int a, b;
      if (X != Y) {
        const int cy = grp[wv][Y + 1] - grp[wv][Y];
        const int u = fchl_div(loc, cy);
        a = grp[wv][X] + u;
        b = grp[wv][Y] + loc - u * cy;
      } else {
        const int cx = grp[wv][X + 1] - grp[wv][X];
        const int u = fchl_pair_row(loc, cx);
        a = grp[wv][X] + u;
        b = grp[wv][X] + u + 1 + (loc - u * (2 * cx - u - 1) / 2);
      }
      const float rij = nr[wv][a], rik = nr[wv][b];
      const float jx = nx[wv][b] - nx[wv][a], jy = ny[wv][b] - ny[wv][a], jz = nz[wv][b] - nz[wv][a];
      const float rjk = sqrtf(jx * jx + jy * jy + jz * jz);
      const float iij = ni[wv][a], iik = ni[wv][b], ijk = fchl_rcp(rjk);
      const float cos_i = (nx[wv][a] * nx[wv][b] + ny[wv][a] * ny[wv][b] + nz[wv][a] * nz[wv][b]) * (iij * iik);
      const float cos_j = -(nx[wv][a] * jx + ny[wv][a] * jy + nz[wv][a] * jz) * (iij * ijk);
      const float cos_k = (nx[wv][b] * jx + ny[wv][b] * jy + nz[wv][b] * jz) * (iik * ijk);
      const float sin_i = sqrtf(fmaxf(0.0f, 1.0f - cos_i * cos_i));
      const float w = c3w * (1.0f + 3.0f * cos_i * cos_j * cos_k) * (nw[wv][a] * nw[wv][b]) *
                      (__builtin_amdgcn_exp2f(-p.N3 * __builtin_amdgcn_logf(rjk)) *
                       fchl_fcut(rjk, rc));
      const int sl = q - q0;
      pw[wv][sl] = make_float2(w * cos_i, w * sin_i);
      pmid[wv][sl] = 0.5f * (rij + rik);
    }
    // element pairs without pairs in the first chunk: their bins start at 0
    if (q0 == 0)
      for (int t = lane; t < NP * p.n3; t += 64) {
        const int Q = fchl_div(t, p.n3);
        const int32_t s0 = seg[wv][Q], s1 = seg[wv][Q + 1] < q1 ? seg[wv][Q + 1] : q1;
        if (s1 <= s0) {
          out3[2 * t] = 0.0f;
          out3[2 * t + 1] = 0.0f;
        }
      }
    wave_sync_lds();
    const int32_t L = q1 - q0;
    int pend = -1;                      // element pair to finish after the tails are stored
    float pc = 0.f, ps = 0.f;
    for (int k = kl; k < p.n3 && g < G; k += 64) {
      const float Rk = rc * float(k) / float(p.n3 - 1);
      const int32_t lo = q0 + fchl_div(L * g, G), hi = q0 + fchl_div(L * (g + 1), G);
      int Q = 0;
      while (Q < NP && seg[wv][Q + 1] <= lo) ++Q;
      bool started = Q < NP && (seg[wv][Q] > q0 ? seg[wv][Q] : q0) >= lo;
      float c = 0.f, sn = 0.f;
      int32_t segend = Q < NP && seg[wv][Q + 1] < q1 ? seg[wv][Q + 1] : q1;
      // one pair a step for every group, whatever their element pairs' ends
      for (int32_t q = lo; q < hi; ++q) {
        const float2 w = pw[wv][q - q0];
        const float d = pmid[wv][q - q0] - Rk;
        const float gk = __builtin_amdgcn_exp2f(keta * (d * d));
        c = __builtin_fmaf(w.x, gk, c);
        sn = __builtin_fmaf(w.y, gk, sn);
        if (q + 1 == segend) {          // element pair Q ends in this part
          if (started) {
            float* o = out3 + 2 * (int64_t(Q) * p.n3 + k);
            if (q0 == 0) {
              o[0] = c;
              o[1] = sn;
            } else {
              o[0] += c;
              o[1] += sn;
            }
          } else {
            pend = Q;
            pc = c;
            ps = sn;
          }
          c = 0.f;
          sn = 0.f;
          ++Q;
          while (Q < NP && seg[wv][Q + 1] <= segend) ++Q;
          started = true;
          segend = Q < NP && seg[wv][Q + 1] < q1 ? seg[wv][Q + 1] : q1;
        }
      }
      tail[wv][lane][0] = c;            // open partial at the end of the part (0 if none)
      tail[wv][lane][1] = sn;
    }
    wave_sync_lds();
    if (pend >= 0) {
      const int32_t st = seg[wv][pend] > q0 ? seg[wv][pend] : q0;
      int gs = g - 1;                   // the group in whose part the element pair starts
      while (gs > 0 && q0 + fchl_div(L * gs, G) > st) --gs;
      float sc = 0.f, ss = 0.f;
      for (int gg = gs; gg < g; ++gg) {
        sc += tail[wv][gg * p.n3 + kl][0];
        ss += tail[wv][gg * p.n3 + kl][1];
      }
      float* o = out3 + 2 * (int64_t(pend) * p.n3 + kl);
      if (q0 == 0) {
        o[0] = sc + pc;
        o[1] = ss + ps;
      } else {
        o[0] += sc + pc;
        o[1] += ss + ps;
      }
    }
    wave_sync_lds();   // weights and tails are reused, and the next chunk adds to these entries
    if (n_pairs == 0) break;
  }
}

// ---------------------------------------------------------------------------
// Coordinate gradient: dR = d(sum_i g_i . rho_i)/dR for an upstream g = dE/drho
// (the forces are -dR). Every three-body term of a centre i and its pair of
// neighbours (j, l) depends on the positions only through the three sides
// a = r_ij, b = r_il, c = r_jl (the cosines follow by the law of cosines), so
// its gradient is dL/da u_ij + dL/db u_il + dL/dc u_jl distributed to the
// three atoms; a two-body term gives dL/dr u_ij to j and minus that to i.
//
// Molecules of at most kFchlSmallAtoms atoms: one workgroup per molecule
// scatters each centre's contributions to its atoms inside LDS. Larger
// molecules: one workgroup per atom gathers the contributions that land on
// it from every centre, so a single large molecule spreads over the chip.
// Every gradient entry is summed in a fixed order (deterministic, no atomics).
// ---------------------------------------------------------------------------
typedef float FchlPair __attribute__((ext_vector_type(2), aligned(4)));

// What a triple needs of one of its sides.
struct FchlSide {
  float r, inv, f, df, pn;   // length, 1 / r, f_cut, d f_cut / dr, r^-N3
};

// dL/da, dL/db, dL/dc for one centre i and neighbour pair (j, l) with sides
// a = r_ij, b = r_il, c = r_jl, where L is the pair's three-body terms
// contracted with the centre's upstream gradient gp (the 2 n3 entries of the
// pair's element pair, [radial bin][cos, sin]). The cosines are functions of
// the sides (law of cosines), so this is the whole positional dependence.
// inv_pn is (a b c)^-N3.
__device__ __forceinline__ void fchl_triple_grad(const FchlSide& sa, const FchlSide& sb,
                                                 const FchlSide& sc, float inv_pn,
                                                 const float* __restrict__ gp,
                                                 const FchlParams& p, float angw, float (&dL)[3]) {
  const float rc = p.rcut;
  const float a = sa.r, b = sb.r, c = sc.r;
  const float ia = sa.inv, ib = sb.inv, ic = sc.inv;
  const float a2 = a * a, b2 = b * b, c2 = c * c;
  const float ci_ = 0.5f * (a2 + b2 - c2) * ia * ib;
  const float cj_ = 0.5f * (a2 + c2 - b2) * ia * ic;
  const float cl_ = 0.5f * (b2 + c2 - a2) * ib * ic;
  const float dci[3] = {0.5f * (a2 - b2 + c2) * ia * ia * ib, 0.5f * (b2 - a2 + c2) * ia * ib * ib,
                        -c * ia * ib};
  const float dcj[3] = {0.5f * (a2 - c2 + b2) * ia * ia * ic, -b * ia * ic,
                        0.5f * (c2 - a2 + b2) * ia * ic * ic};
  const float dcl[3] = {-a * ib * ic, 0.5f * (b2 - c2 + a2) * ib * ib * ic,
                        0.5f * (c2 - b2 + a2) * ib * ic * ic};
  const float si = sqrtf(fmaxf(0.0f, 1.0f - ci_ * ci_));
  const float dsi_dc = si > 1e-12f ? -ci_ * fchl_rcp(si) : 0.0f;
  const float C = ci_ * cj_ * cl_;
  const float invP3 = inv_pn;
  const float xi3 = p.c3 * (1.0f + 3.0f * C) * invP3;
  const float fa = sa.f, fb = sb.f, fcc = sc.f;
  const float dfa = sa.df, dfb = sb.df, dfcc = sc.df;
  const float Fc = fa * fb * fcc;
  const float dF[3] = {dfa * fb * fcc, fa * dfb * fcc, fa * fb * dfcc};
  const float inv_side[3] = {ia, ib, ic};
  const float A = angw * xi3 * Fc;
  const float wc = A * ci_, ws = A * si;
  const float mid = 0.5f * (a + b);
  const float step = rc / float(p.n3 - 1);
  // radial bins: rad = exp(-eta3 d^2), d rad / d mid = -2 eta3 d rad
  const float keta = -p.eta3 * 1.44269504088896341f;
  float Gc = 0.f, Gs = 0.f, Gcp = 0.f, Gsp = 0.f;
#pragma unroll 4
  for (int k = 0; k < p.n3; ++k) {
    const FchlPair g = *reinterpret_cast<const FchlPair*>(gp + 2 * k);
    const float d = mid - float(k) * step;
    const float rad = __builtin_amdgcn_exp2f(keta * (d * d));
    const float drad = d * rad;
    Gc = __builtin_fmaf(g.x, rad, Gc);
    Gs = __builtin_fmaf(g.y, rad, Gs);
    Gcp = __builtin_fmaf(g.x, drad, Gcp);
    Gsp = __builtin_fmaf(g.y, drad, Gsp);
  }
  Gcp *= -2.0f * p.eta3;
  Gsp *= -2.0f * p.eta3;
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const float dC = dci[v] * cj_ * cl_ + ci_ * dcj[v] * cl_ + ci_ * cj_ * dcl[v];
    const float dxi = p.c3 * 3.0f * dC * invP3 - p.N3 * xi3 * inv_side[v];
    const float dA = angw * (dxi * Fc + xi3 * dF[v]);
    const float dwc = dA * ci_ + A * dci[v];
    const float dws = dA * si + A * dsi_dc * dci[v];
    const float dmid = v < 2 ? 0.5f : 0.0f;
    dL[v] = Gc * dwc + Gs * dws + (wc * Gcp + ws * Gsp) * dmid;
  }
}

// A side from its length alone (r^-N3 left out).
__device__ __forceinline__ FchlSide fchl_side(float r, const FchlParams& p) {
  return FchlSide{r, fchl_rcp(r), fchl_fcut(r, p.rcut), fchl_dfcut(r, p.rcut), 0.0f};
}

// d/dr of the two-body terms of one neighbour at distance r, contracted with
// the centre's upstream gradient gX (the n2 bins of the neighbour's element),
// over the bins k0, k0 + kstep, ...
__device__ __forceinline__ float fchl_pair_grad(float r, const float* __restrict__ gX,
                                                const FchlParams& p, int k0 = 0, int kstep = 1) {
  const float rc = p.rcut;
  const float q = 1.0f + p.eta2 / (r * r);
  const float s2 = logf(q);
  const float ds2 = -2.0f * p.eta2 / (r * r * r * q);
  const float mu = logf(r / sqrtf(q));
  const float dmu = 1.0f / r + p.eta2 / (r * r * r * q);
  const float fcv = fchl_fcut(r, rc);
  const float dfc = fchl_dfcut(r, rc);
  const float pref = powf(r, -p.N2) / (sqrtf(s2) * 2.50662827463100f);
  const float is2 = 1.0f / s2;
  // D = D0 + Lk D1 + Lk^2 D2
  const float D0 = -p.N2 / r - 0.5f * ds2 * is2, D1 = dmu * is2, D2 = 0.5f * ds2 * is2 * is2;
  const float step = rc / float(p.n2);
  float dL = 0.0f;
  for (int k = k0; k < p.n2; k += kstep) {
    const float Rk = float(k + 1) * step;
    const float Lk = fchl_ln(Rk) - mu;
    const float B = pref * fchl_exp(-0.5f * Lk * Lk * is2) * fchl_rcp(Rk);
    const float D = D0 + Lk * (D1 + Lk * D2);
    dL += gX[k] * (dfc + fcv * D) * B;
  }
  return dL;
}

// Molecules of at most kFchlSmallAtoms atoms: one workgroup per molecule,
// its NW waves take NW centres at a time. For a centre with n
// neighbours, every unordered pair is evaluated once: lanes take the pairs
// (in chunks of kFchlBwdPairs) and store dL/da, dL/db, dL/dc in the wave's
// LDS (dL/dc over r_st). Then each neighbour s gets H lanes (H = 4, 2, 1 for at most 16, 32,
// 63 neighbours); lane h walks the partners t = h, h + H, ... in order (and
// the two-body bins h, h + H, ...) and sums T_s (dL/da where s is the pair's
// j, dL/db where it is l, plus its two-body term) and V_s = -sum dL/dc
// (x_t - x_s) / r_st; the H parts are combined by fixed shuffles. Neighbour s
// gets T_s u_s + V_s, the centre -sum_s T_s u_s (u_s the unit vector from the
// centre to s, summed by fixed shuffles), and the centres' results are
// merged into the molecule's gradient in centre order, so the bits do not
// depend on NW. NW = 4 fills the chip with four molecules to a compute unit;
// up to kFchlFewMols molecules each has a compute unit to itself, and NW = 16
// shortens its chain (21 atoms: 66 us with four waves, 35 with 16).
// STAGED: the centre's upstream gradient row (at most kFchlStage entries) is
// copied into the wave's LDS first, so that the radial-bin loops read LDS.
constexpr int kFchlSmallAtoms = 64;
constexpr int kFchlFewMols = 256;   // molecules that take 16 waves each
constexpr int kFchlStage = 1024;
constexpr int kFchlBwdPairs = 256;

template <bool STAGED, int NW>
__global__ __launch_bounds__(64 * NW) void fchl19_backward_small_kernel(
    const float* __restrict__ R, const int32_t* __restrict__ element,
    const int64_t* __restrict__ mol_ptr, int64_t m0, int64_t n_mols, int32_t E, FchlParams p,
    int64_t size, const float* __restrict__ g, float* __restrict__ dR) {
  __shared__ float ax[kFchlSmallAtoms], ay[kFchlSmallAtoms], az[kFchlSmallAtoms];
  __shared__ int32_t ael[kFchlSmallAtoms];
  __shared__ float gsum[3][kFchlSmallAtoms];
  __shared__ float res[NW][3][kFchlSmallAtoms];
  __shared__ int32_t nid[NW][kFchlSmallAtoms];
  __shared__ float dls[NW][3][kFchlBwdPairs];
  __shared__ float gst[NW][STAGED ? kFchlStage : 1];
  __shared__ float4 side[NW][kFchlSmallAtoms];   // r, 1 / r, f_cut, its derivative

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t m = m0 + blockIdx.x;
  if (m >= n_mols) return;
  const int64_t a0 = mol_ptr[m];
  const int N = int(mol_ptr[m + 1] - a0);
  if (N <= 0 || N > kFchlSmallAtoms) return;   // larger molecules: fchl19_backward_gather_kernel
  const float rc = p.rcut;
  if (tid < N) {
    ax[tid] = R[3 * (a0 + tid)];
    ay[tid] = R[3 * (a0 + tid) + 1];
    az[tid] = R[3 * (a0 + tid) + 2];
    ael[tid] = element[a0 + tid];
    gsum[0][tid] = gsum[1][tid] = gsum[2][tid] = 0.0f;
  }
  __syncthreads();
  const float angw = 2.0f * expf(-0.5f * p.zeta * p.zeta) * sqrtf(p.eta3 / 3.14159265358979f);

  for (int c0 = 0; c0 < N; c0 += NW) {
    const int ci = c0 + wv;
    res[wv][0][lane] = res[wv][1][lane] = res[wv][2][lane] = 0.0f;
    if (ci < N) {   // wave-uniform
      const float* __restrict__ gi = g + (a0 + ci) * size;
      if (STAGED) {
        for (int64_t t = lane; t < size; t += 64) gst[wv][t] = gi[t];
        gi = &gst[wv][0];   // made visible by the wave barrier below
      }
      const float xi = ax[ci], yi = ay[ci], zi = az[ci];
      // this lane's candidate atom, then the neighbours in element order
      const int t = lane;
      bool in = false;
      if (t < N && t != ci) {
        const float dx = ax[t] - xi, dy = ay[t] - yi, dz = az[t] - zi;
        in = sqrtf(dx * dx + dy * dy + dz * dz) < rc;
      }
      int n = 0;
      for (int X = 0; X < E; ++X) {
        const bool f = in && ael[t < N ? t : 0] == X;
        const uint64_t mask = __ballot(f);
        if (f) nid[wv][n + __popcll(mask & ((uint64_t(1) << lane) - 1))] = t;
        n += __popcll(mask);
      }
      wave_sync_lds();
      if (lane < n) {   // lane = slot here: what the pairs need of one neighbour alone
        const int j = nid[wv][lane];
        const float vx = ax[j] - xi, vy = ay[j] - yi, vz = az[j] - zi;
        const float r = sqrtf(vx * vx + vy * vy + vz * vz);
        side[wv][lane] = make_float4(r, fchl_rcp(r), fchl_fcut(r, rc), fchl_dfcut(r, rc));
      }
      wave_sync_lds();
      // H lanes per neighbour slot when the neighbours are few: lane (sl, h)
      // takes the two-body bins and the partners h, h + H, ... of slot sl
      const int H = n <= 16 ? 4 : (n <= 32 ? 2 : 1);
      const int sl = lane / H, h = lane % H;
      int js = 0;
      float xs = 0.f, ys = 0.f, zs = 0.f, ux = 0.f, uy = 0.f, uz = 0.f;
      float T = 0.f, Vx = 0.f, Vy = 0.f, Vz = 0.f;
      if (sl < n) {
        js = nid[wv][sl];
        xs = ax[js];
        ys = ay[js];
        zs = az[js];
        const float vx = xs - xi, vy = ys - yi, vz = zs - zi;
        const float rs = sqrtf(vx * vx + vy * vy + vz * vz);
        ux = vx / rs;
        uy = vy / rs;
        uz = vz / rs;
        T = fchl_pair_grad(rs, gi + ael[js] * p.n2, p, h, H);
      }
      const int32_t n_pairs = n * (n - 1) / 2;
      for (int32_t q0 = 0; q0 < n_pairs; q0 += kFchlBwdPairs) {
        const int32_t q1 = q0 + kFchlBwdPairs < n_pairs ? q0 + kFchlBwdPairs : n_pairs;
        for (int32_t q = q0 + lane; q < q1; q += 64) {
          // q -> slots (s, t), s < t; row s starts at s (2n - s - 1) / 2
          const float c2n = 2.0f * float(n) - 1.0f;
          int s = int((c2n - sqrtf(c2n * c2n - 8.0f * float(q))) * 0.5f);
          s = s < 0 ? 0 : (s > n - 2 ? n - 2 : s);
          while (s > 0 && s * (2 * n - s - 1) / 2 > q) --s;
          while ((s + 1) * (2 * n - s - 2) / 2 <= q) ++s;
          const int tt = s + 1 + (q - s * (2 * n - s - 1) / 2);
          const int ja = nid[wv][s], jb = nid[wv][tt];
          const float vax = ax[ja] - xi, vay = ay[ja] - yi, vaz = az[ja] - zi;
          const float vbx = ax[jb] - xi, vby = ay[jb] - yi, vbz = az[jb] - zi;
          const float4 fa = side[wv][s], fb = side[wv][tt];
          const float wx = vbx - vax, wy = vby - vay, wz = vbz - vaz;
          const float c = sqrtf(wx * wx + wy * wy + wz * wz);
          const int Xa = ael[ja], Xb = ael[jb];
          const int P = fchl_pair(Xa < Xb ? Xa : Xb, Xa < Xb ? Xb : Xa, E);
          const FchlSide A{fa.x, fa.y, fa.z, fa.w, 0.0f}, B{fb.x, fb.y, fb.z, fb.w, 0.0f};
          const FchlSide C = fchl_side(c, p);
          float dL[3];
          fchl_triple_grad(A, B, C,
                           __builtin_amdgcn_exp2f(-p.N3 * __builtin_amdgcn_logf(fa.x * fb.x * c)),
                           gi + int64_t(E) * p.n2 + int64_t(P) * p.n3 * 2, p, angw, dL);
          const int sl = q - q0;
          dls[wv][0][sl] = dL[0];
          dls[wv][1][sl] = dL[1];
          dls[wv][2][sl] = dL[2] * C.inv;
        }
        wave_sync_lds();
        if (sl < n) {
          const int s = sl;
          for (int u = h; u < n; u += H) {
            if (u == s) continue;
            const int lo = s < u ? s : u, hi = s < u ? u : s;
            const int32_t q = lo * (2 * n - lo - 1) / 2 + (hi - lo - 1);
            if (q < q0 || q >= q1) continue;
            const int sl = q - q0;
            T += s < u ? dls[wv][0][sl] : dls[wv][1][sl];
            const int ju = nid[wv][u];
            const float wx = ax[ju] - xs, wy = ay[ju] - ys, wz = az[ju] - zs;
            const float f = dls[wv][2][sl];
            Vx -= f * wx;
            Vy -= f * wy;
            Vz -= f * wz;
          }
        }
        wave_sync_lds();   // the chunk's derivatives are no longer read
      }
      // the H parts of a slot, combined in a fixed order (every lane of the
      // slot then holds the same sums)
      if (H >= 2) {
        T += __shfl_xor(T, 1);
        Vx += __shfl_xor(Vx, 1);
        Vy += __shfl_xor(Vy, 1);
        Vz += __shfl_xor(Vz, 1);
      }
      if (H >= 4) {
        T += __shfl_xor(T, 2);
        Vx += __shfl_xor(Vx, 2);
        Vy += __shfl_xor(Vy, 2);
        Vz += __shfl_xor(Vz, 2);
      }
      const bool owner = sl < n && h == 0;
      if (owner) {
        res[wv][0][js] = T * ux + Vx;
        res[wv][1][js] = T * uy + Vy;
        res[wv][2][js] = T * uz + Vz;
      }
      // the centre's total over the slots' owner lanes, in a fixed butterfly order
      float cx = owner ? -T * ux : 0.f, cy = owner ? -T * uy : 0.f, cz = owner ? -T * uz : 0.f;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        cx += __shfl_xor(cx, o);
        cy += __shfl_xor(cy, o);
        cz += __shfl_xor(cz, o);
      }
      if (lane == 0) {
        res[wv][0][ci] = cx;
        res[wv][1][ci] = cy;
        res[wv][2][ci] = cz;
      }
    }
    __syncthreads();
    if (tid < N) {
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        float acc = gsum[v][tid];
#pragma unroll
        for (int w = 0; w < NW; ++w) acc += res[w][v][tid];
        gsum[v][tid] = acc;
      }
    }
    __syncthreads();
  }
  if (tid < N) {
    dR[3 * (a0 + tid)] = gsum[0][tid];
    dR[3 * (a0 + tid) + 1] = gsum[1][tid];
    dR[3 * (a0 + tid) + 2] = gsum[2][tid];
  }
}

// Molecules above kFchlSmallAtoms atoms (any size): one workgroup per atom
// t gathers the gradient at R_t from every centre whose representation
// depends on it, t itself and each neighbour c of t:
//   centre t: -dL/dr (R_s - R_t) / r_ts for the two-body term of every
//     neighbour s, and -(dL/da (R_j - R_t) / a + dL/db (R_l - R_t) / b) for
//     every unordered neighbour pair {j, l} (a = r_tj, b = r_tl);
//   centre c: dL/dr (R_t - R_c) / r_ct for t's two-body term, and for every
//     other neighbour l of c the pair {t, l}, with sides a = r_ct, b = r_cl,
//     c = r_tl: dL/da (R_t - R_c) / a + dL/dc (R_t - R_l) / c.
// The three-body terms are symmetric in the pair's two atoms (the mean
// distance, the centre's angle and the product of the three cosines do not
// change when j and l swap), so the pair's sides may be passed in either
// order. t's neighbours are gathered into LDS as in the forward kernel
// (kFchlMaxNb at most; more leave t's row NaN). A pair {t, l} of a centre c
// carries f_cut(r_tl), so l is itself a neighbour of t: the centre-c terms
// come from the pairs (c, l) of t's own list with r_cl < r_cut. Each thread
// sums a fixed subset of the terms and the threads' sums are added in thread
// order: the result is deterministic and does not depend on the rest of the
// batch; the sums are FP64, since an atom of a large molecule gathers
// thousands of terms. Every pair derivative of a centre is evaluated once for
// each of the pair's atoms (three times over), the price of needing no
// workspace and no bound on the molecule's size.
//
// Bound by vector issue, about 350 instructions a triple, most of them the
// radial bins. 16 waves to a workgroup, so that a compute unit with one atom
// has four on each SIMD; what depends on one neighbour alone (1 / r, f_cut
// and its derivative, r^-N3) is formed once per neighbour. 124 us for the 245
// atoms of a cluster with four waves and every factor formed per triple, now 47.
template <int NT>
__device__ __forceinline__ void fchl19_backward_atom(int64_t t, int64_t a0, int64_t a1,
                                     const float* __restrict__ R,
                                     const int32_t* __restrict__ element, int32_t E,
                                     const FchlParams& p, int64_t size,
                                     const float* __restrict__ g, float* __restrict__ dR) {
  constexpr int VT = kFchlThreads, NW = VT / 64;   // sums of VT threads, whatever NT
  __shared__ int32_t nidx[kFchlMaxNb];
  __shared__ float nx[kFchlMaxNb], ny[kFchlMaxNb], nz[kFchlMaxNb];
  __shared__ FchlSide ns[kFchlMaxNb];
  __shared__ FchlGather<NT> gathered;
  __shared__ int32_t seg[kFchlMaxElements * (kFchlMaxElements + 1) / 2 + 1];
  __shared__ int32_t pair_xy[kFchlMaxElements * (kFchlMaxElements + 1) / 2];
  __shared__ double red[3][NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const float rc = p.rcut;
  const float angw = 2.0f * expf(-0.5f * p.zeta * p.zeta) * sqrtf(p.eta3 / 3.14159265358979f);
  const int NP = E * (E + 1) / 2;
  const int et = element[t];
  const int32_t* const grp = gathered.grp;
  const int total = fchl_gather<NT>(
      t, a0, a1, R, element, E, rc, gathered,
      [&](int sl, int64_t j, float dx, float dy, float dz, float r) {
        nidx[sl] = int32_t(j - a0);
        nx[sl] = dx;
        ny[sl] = dy;
        nz[sl] = dz;
        ns[sl] = FchlSide{r, fchl_rcp(r), fchl_fcut(r, rc), fchl_dfcut(r, rc), powf(r, -p.N3)};
      });
  const bool bad = total > kFchlMaxNb;   // uniform: every thread counted the same chunks
  if (!bad) {
    fchl_segments<NT>(grp, E, seg, pair_xy);
    __syncthreads();
    const float* __restrict__ gt = g + t * size;
    // a triple whose sides a and b end at t and whose third side is new
    const auto far_side = [&](float r) {
      return FchlSide{r, fchl_rcp(r), fchl_fcut(r, rc), fchl_dfcut(r, rc),
                      __builtin_amdgcn_exp2f(-p.N3 * __builtin_amdgcn_logf(r))};
    };
    const int32_t n_pairs = seg[NP], n_cl = total * total;
    for (int vt = tid; vt < VT; vt += NT) {
      double px = 0.0, py = 0.0, pz = 0.0;   // FP64 sums: a large centre adds thousands of terms
      if (vt - lane < max(n_pairs, n_cl)) {  // a wave with terms
        // centre t, two-body
        for (int sl = vt; sl < total; sl += VT) {
          int X = 0;
          while (sl >= grp[X + 1]) ++X;
          const float f = fchl_pair_grad(ns[sl].r, gt + X * p.n2, p) * ns[sl].inv;
          px -= f * nx[sl];
          py -= f * ny[sl];
          pz -= f * nz[sl];
        }
        // centre t, three-body over its unordered neighbour pairs
        int P = 0;   // non-decreasing over this thread's pairs
        for (int32_t q = vt; q < n_pairs; q += VT) {
          while (q >= seg[P + 1]) ++P;
          const int X = pair_xy[P] & 255, Y = pair_xy[P] >> 8;
          const int32_t loc = q - seg[P];
          int sa, sb;
          if (X != Y) {
            const int cyn = grp[Y + 1] - grp[Y];
            const int u = fchl_div(loc, cyn);
            sa = grp[X] + u;
            sb = grp[Y] + loc - u * cyn;
          } else {
            const int cxn = grp[X + 1] - grp[X];
            const int u = fchl_pair_row(loc, cxn);
            sa = grp[X] + u;
            sb = grp[X] + u + 1 + (loc - u * (2 * cxn - u - 1) / 2);
          }
          const float wx = nx[sb] - nx[sa], wy = ny[sb] - ny[sa], wz = nz[sb] - nz[sa];
          const float c = sqrtf(wx * wx + wy * wy + wz * wz);
          if (!(c < rc)) continue;   // f_cut(r_jl) and its derivative vanish
          const FchlSide A = ns[sa], B = ns[sb], C = far_side(c);
          float dL[3];
          fchl_triple_grad(A, B, C, A.pn * B.pn * C.pn,
                           gt + int64_t(E) * p.n2 + int64_t(P) * p.n3 * 2, p, angw, dL);
          const float fa = dL[0] * A.inv, fb = dL[1] * B.inv;
          px -= fa * nx[sa] + fb * nx[sb];
          py -= fa * ny[sa] + fb * ny[sb];
          pz -= fa * nz[sa] + fb * nz[sb];
        }
        // each neighbour c of t as a centre: t's two-body term in c's row, and
        // the pairs {t, l} of c. A pair's terms carry f_cut(r_tl), so only the
        // neighbours l of t contribute, and those are in t's list: the pairs
        // (c, l) of t's list with r_cl < r_cut, flattened over the threads
        for (int cs = vt; cs < total; cs += VT) {
          const float* __restrict__ gc = g + (a0 + nidx[cs]) * size;
          const float f = fchl_pair_grad(ns[cs].r, gc + et * p.n2, p) * ns[cs].inv;
          px -= f * nx[cs];   // (R_t - R_c) = -(R_c - R_t)
          py -= f * ny[cs];
          pz -= f * nz[cs];
        }
        for (int32_t q = vt; q < n_cl; q += VT) {
          const int cs = fchl_div(q, total), ls = q - cs * total;
          if (ls == cs) continue;
          const float wx = nx[ls] - nx[cs], wy = ny[ls] - ny[cs], wz = nz[ls] - nz[cs];   // R_l - R_c
          const float rcl = sqrtf(wx * wx + wy * wy + wz * wz);
          if (!(rcl < rc)) continue;
          int Y = 0;
          while (ls >= grp[Y + 1]) ++Y;
          const int Pc = et <= Y ? fchl_pair(et, Y, E) : fchl_pair(Y, et, E);
          const float* __restrict__ gc = g + (a0 + nidx[cs]) * size;
          const FchlSide A = ns[cs], B = far_side(rcl), C = ns[ls];
          float dL[3];
          fchl_triple_grad(A, B, C, A.pn * C.pn * B.pn,
                           gc + int64_t(E) * p.n2 + int64_t(Pc) * p.n3 * 2, p, angw, dL);
          // dL/da (R_t - R_c) / a + dL/dc (R_t - R_l) / c, with R_x - R_t = n[x]
          const float fa = dL[0] * A.inv, fc = dL[2] * C.inv;
          px -= fa * nx[cs] + fc * nx[ls];
          py -= fa * ny[cs] + fc * ny[ls];
          pz -= fa * nz[cs] + fc * nz[ls];
        }
        // lanes in a fixed order
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          px += __shfl_xor(px, o);
          py += __shfl_xor(py, o);
          pz += __shfl_xor(pz, o);
        }
      }
      if (lane == 0) {
        red[0][vt >> 6] = px;
        red[1][vt >> 6] = py;
        red[2][vt >> 6] = pz;
      }
    }
  }
  __syncthreads();
  if (tid < 3) {
    double sum = 0.0;
    for (int k = 0; k < NW; ++k) sum += red[tid][k];
    dR[3 * t + tid] = bad ? __builtin_nanf("") : float(sum);
  }
  __syncthreads();   // red[], the neighbour list and seg[] are rewritten for the next atom
}

// Molecules above kFchlSmallAtoms atoms, dealt out as the forward kernel deals them.
template <int NT>
__global__ __launch_bounds__(NT) void fchl19_backward_gather_kernel(
    const float* __restrict__ R, const int32_t* __restrict__ element,
    const int64_t* __restrict__ mol_ptr, int64_t n_mols, int32_t E, FchlParams p, int64_t size,
    const float* __restrict__ g, float* __restrict__ dR) {
  __shared__ FchlDeal<NT> deal;
  fchl_deal<NT>(mol_ptr, n_mols, kFchlSmallAtoms, deal, [&](int64_t t, int64_t a0, int64_t a1) {
    fchl19_backward_atom<NT>(t, a0, a1, R, element, E, p, size, g, dR);
  });
}

}  // namespace sorf

using namespace sorf;

int64_t sorf_fchl19_len(int32_t E, int32_t n2, int32_t n3) {
  return int64_t(E) * n2 + int64_t(E) * (E + 1) / 2 * n3 * 2;
}

// Workgroups of the kernels for large molecules, all resident so that the size scan runs
// once: of kFchlThreads threads and one per compute unit (registers) while every atom has
// one to itself, of half as many and two per unit (LDS) for more atoms, which hide one's
// barriers and loads behind the other's work (forward and backward, us): 245 atoms with 46
// neighbours 41 and 54, with the halves 52 and 59; 1260 atoms 122 and 151, halves 99 and
// 131; 1000 molecules of 65 atoms with eight neighbours 2376 and 4132, halves 1360 and 2083.
constexpr int64_t kFchlUnits = 256;
static bool fchl_few_atoms(int64_t n_atoms, int32_t n3) {
  return n_atoms <= kFchlUnits || n3 > kFchlThreads / 2;
}

hipError_t sorf_launch_fchl19_forward(const float* R, const int32_t* element,
                                      const int64_t* mol_ptr, int64_t n_atoms, int64_t n_mols,
                                      int32_t E, const FchlParamsHost& ph, float* rho,
                                      hipStream_t st) {
  if (n_atoms == 0) return hipSuccess;
  const FchlParams p{ph.n2, ph.n3, ph.eta2, ph.eta3, ph.N2, ph.N3, ph.c3, ph.zeta, ph.rcut};
  const int64_t size = sorf_fchl19_len(E, ph.n2, ph.n3);
  constexpr int64_t kPerLaunch = int64_t(1) << 30;
  for (int64_t a0 = 0; a0 < n_atoms; a0 += kPerLaunch) {
    const int64_t cnt = n_atoms - a0 < kPerLaunch ? n_atoms - a0 : kPerLaunch;
    hipLaunchKernelGGL(fchl19_forward_small_kernel, dim3(unsigned((cnt + 3) / 4)), dim3(256), 0, st,
                       R, element, mol_ptr, a0, n_atoms, n_mols, E, p, size, rho);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (n_mols == 0) return hipSuccess;
  const auto go = [&](auto kernel, int threads, int64_t most) {
    hipLaunchKernelGGL(kernel, dim3(unsigned(n_atoms < most ? n_atoms : most)), dim3(unsigned(threads)),
                       0, st, R, element, mol_ptr, n_mols, E, p, size, rho);
  };
  if (fchl_few_atoms(n_atoms, ph.n3))
    go(fchl19_forward_kernel<kFchlThreads>, kFchlThreads, kFchlUnits);
  else
    go(fchl19_forward_kernel<kFchlThreads / 2>, kFchlThreads / 2, 2 * kFchlUnits);
  return hipGetLastError();
}

hipError_t sorf_launch_fchl19_backward(const float* R, const int32_t* element,
                                       const int64_t* mol_ptr, int64_t n_atoms, int64_t n_mols,
                                       int32_t E, const FchlParamsHost& ph, const float* g, float* dR,
                                       hipStream_t st) {
  if (n_mols == 0) return hipSuccess;
  const FchlParams p{ph.n2, ph.n3, ph.eta2, ph.eta3, ph.N2, ph.N3, ph.c3, ph.zeta, ph.rcut};
  const int64_t size = sorf_fchl19_len(E, ph.n2, ph.n3);
  constexpr int64_t kPerLaunch = int64_t(1) << 30;
  for (int64_t m0 = 0; m0 < n_mols; m0 += kPerLaunch) {
    const int64_t cnt = n_mols - m0 < kPerLaunch ? n_mols - m0 : kPerLaunch;
    const auto go = [&](auto kernel, unsigned threads) {
      hipLaunchKernelGGL(kernel, dim3(unsigned(cnt)), dim3(threads), 0, st, R, element, mol_ptr,
                         m0, n_mols, E, p, size, g, dR);
    };
    const bool few = n_mols <= kFchlFewMols;
    if (size <= kFchlStage && few)
      go(fchl19_backward_small_kernel<true, 16>, 1024);
    else if (size <= kFchlStage)
      go(fchl19_backward_small_kernel<true, 4>, 256);
    else if (few)
      go(fchl19_backward_small_kernel<false, 16>, 1024);
    else
      go(fchl19_backward_small_kernel<false, 4>, 256);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // molecules above kFchlSmallAtoms atoms
  const auto go = [&](auto kernel, int threads, int64_t most) {
    hipLaunchKernelGGL(kernel, dim3(unsigned(n_atoms < most ? n_atoms : most)), dim3(unsigned(threads)),
                       0, st, R, element, mol_ptr, n_mols, E, p, size, g, dR);
  };
  if (fchl_few_atoms(n_atoms, ph.n3))
    go(fchl19_backward_gather_kernel<kFchlThreads>, kFchlThreads, kFchlUnits);
  else
    go(fchl19_backward_gather_kernel<kFchlThreads / 2>, kFchlThreads / 2, 2 * kFchlUnits);
  return hipGetLastError();
}
