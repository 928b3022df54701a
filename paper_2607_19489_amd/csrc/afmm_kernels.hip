// HIP kernels of the adaptive FMM for gfx950.
//
// Group = the 8 children of one refined cell F.  The 8 siblings share F's
// interaction list (Sec. 2): the level-(f-1) cells of the 6^3 block around
// F's oct minus the 27 cells touching F, i.e. the children of the 27
// neighbours of F's father G minus F's own neighbours.  Relative to F the
// source offsets d = s - F form a fixed set of 189 "taps" that depends only on
// F's octant (parity class), and the translation operator of a tap depends
// only on d and the child octant.  Groups of one parity class therefore share
// every operator: M2L and the intermediate-field M2P become, tap by tap, dense
// products  OUT[rows x groups] += A_d[rows x K] * S[K x groups]  on MFMA.
//
// Deterministic: every sum runs in a fixed order.  The only atomics number the fathers
// of an M2P tile in LDS; their places do not show in the results.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>

#include "afmm_internal.h"
#include "afmm_mfma.h"

namespace afmm {

namespace {

constexpr int kBlock = 256;
constexpr int kTaps = 189;

inline int ceil_div_host(int a, int b) { return (a + b - 1) / b; }

__device__ inline int e_axis(int e, int d) { return (d == 0 ? e % 3 : (d == 1 ? (e / 3) % 3 : e / 9)) - 1; }
__device__ inline int o_axis(int o, int d) { return (o >> d) & 1; }
__device__ inline int d_index(int dx, int dy, int dz) { return (dx + 3) + 7 * (dy + 3) + 49 * (dz + 3); }

template <typename T>
__device__ inline T rsqrt_t(T x);
template <>
__device__ inline float rsqrt_t<float>(float x) { return rsqrtf(x); }
template <>
__device__ inline double rsqrt_t<double>(double x) { return 1.0 / sqrt(x); }

// P2P in target-level units: phi~ -= m/|R|, a~ -= m R/|R|^3.
template <typename T>
__device__ inline void p2p(T rx, T ry, T rz, T m, T* out) {
  const T r2 = rx * rx + ry * ry + rz * rz;
  const T inv = rsqrt_t<T>(r2);
  const T w = m * inv;
  const T w3 = w * inv * inv;
  out[0] -= w;
  out[1] -= w3 * rx;
  out[2] -= w3 * ry;
  out[3] -= w3 * rz;
}

// Compile-time tables of the folded coefficients of order P: degree, position
// in the full order, and the full position of a + e_i (or -1 when |a| = P).
template <int P>
struct HTab {
  int deg[nh(P)];
  int full[nh(P)];
  int up[nh(P)][3];
  constexpr HTab() : deg(), full(), up() {
    for (int n = 0; n <= P; ++n)
      for (int c = 0; c <= (n > 0 ? 1 : 0); ++c)
        for (int b = 0; b <= n - c; ++b) {
          const int a = n - b - c, h = h_index(a, b, c);
          deg[h] = n;
          full[h] = mi_index(a, b, c);
          for (int i = 0; i < 3; ++i)
            up[h][i] = n < P ? mi_index(a + (i == 0), b + (i == 1), c + (i == 2)) : -1;
        }
  }
};

// M2P of one multipole with a D~ row, for the near field (VALU): fully
// unrolled over the folded coefficients, so every D~ and source index (and the
// weight 2^-|a| of the same-level source copy) is a compile-time constant.
template <typename T, int P>
__device__ inline void m2p_row(const T* __restrict__ D, const T* __restrict__ S, T* out) {
  constexpr int K = nh(P);
  constexpr int K1 = nh(P - 1);
  constexpr HTab<P> mt{};
  constexpr SymLayout<P, (int)sizeof(T)> sl{};
  T phi = 0, ax = 0, ay = 0, az = 0;
#pragma unroll
  for (int a = 0; a < K1; ++a) {
    const T w = (T)(1.0 / (double)(1 << mt.deg[a])) * S[sl.pos[a]];
    phi += w * D[mt.full[a]];
    ax += w * D[mt.up[a][0]];
    ay += w * D[mt.up[a][1]];
    az += w * D[mt.up[a][2]];
  }
#pragma unroll
  for (int a = K1; a < K; ++a) phi += (T)(1.0 / (double)(1 << mt.deg[a])) * S[sl.pos[a]] * D[mt.full[a]];
  out[0] += phi;
  out[1] -= ax;
  out[2] -= ay;
  out[3] -= az;
}

}  // namespace

// ---------------------------------------------------------------------------
// leaf masses of one level (slot gather); refined cells get 0
__global__ void k_gather_mass(int n, const int32_t* __restrict__ rank, const int32_t* __restrict__ slot,
                              const double* __restrict__ m, double* __restrict__ out, double* __restrict__ snap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int s = slot[i];
  const double v = s >= 0 ? m[s] : 0.0;
  out[i] = rank[i] < 0 ? v : 0.0;
  if (snap && s >= 0) snap[s] = v;
}

hipError_t launch_gather_mass(const LevelDev& lv, const double* m_src, double* snap, hipStream_t st) {
  if (lv.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_mass, dim3(ceil_div_host(lv.n, 256)), dim3(256), 0, st, lv.n, lv.rank, lv.slot,
                     m_src, lv.mass, snap);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Folded source copies of the nc cells of a block (256 threads): cell c's row
// index by rank(c), its folded coefficient h by coef(c, h); written slot by slot
// in row order, so consecutive threads store consecutive addresses (0 in the
// padding slots).
template <int P, typename Rank, typename Coef>
__device__ inline void store_copies(int nc, const LevelDev& lv, Rank rank, Coef coef) {
  constexpr int R32 = src_row(P, 4), R64 = src_row(P, 8);
  static constexpr SymLayout<P, 4> l32{};
  static constexpr SymLayout<P, 8> l64{};
  if (lv.S32)
    for (int i = threadIdx.x; i < nc * R32; i += 256) {
      const int c = i / R32, sl = i - c * R32, h = l32.coef[sl];
      lv.S32[(size_t)rank(c) * R32 + sl] = h >= 0 ? (float)coef(c, h) : 0.f;
    }
  if (lv.Sc64)
    for (int i = threadIdx.x; i < nc * R64; i += 256) {
      const int c = i / R64, sl = i - c * R64, h = l64.coef[sl];
      lv.Sc64[(size_t)rank(c) * R64 + sl] = h >= 0 ? coef(c, h) : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Upward pass (Alg. 2 Upward + CenterShift), FP64.  With child offsets
// d_o = (o - 1/2)/2 the M2M weight C(a,k) d_o^(a-k) 2^-|k| splits into
// C(a,k) 4^-|a-k| 2^-|k| times a sign that depends only on the parity of
// a - k, so the 8 children are first folded into 8 signed sums per
// coefficient:  Y[k][q] = sum_o (prod_{i: q_i=1} sgn(o_i)) S_o[k].
// The weights C(a,k) 4^-|a-k| 2^-|k| and signs are tabulated per coefficient a
// (cm.m2m_list: for each a, its (k, parity) entries; cm.m2m_w the weights).
// Thread = (cell, coefficient) over chunks of CB cells; a block is persistent:
// it stages the entry tables in LDS once, then for each chunk loads the
// children's ranks and masses, forms the 8 signed child sums Y of each cell in
// LDS and sums the entries of each coefficient.
// The coefficients then go to LDS, from where the folded source copies are
// formed slot by slot of their layout (0 in the padding slots).  Runs
// over a list of the level's refined ranks (those with a refined child;
// k_p2m_leaf takes the others).
// Cells per chunk: as many as fit the block, at most 32 (one child per thread in
// the loads).
__host__ __device__ constexpr int upward_cells(int p) { return 256 / nmi(p) < 32 ? 256 / nmi(p) : 32; }

// entries of the fold lists (CommonDev::fold_list)
__host__ __device__ constexpr int fold_entries(int p) {
  int n = 0;
  for (int d = 0; d <= p; ++d)
    for (int z = 0; z <= (d > 0 ? 1 : 0); ++z)
      for (int b = 0; b <= d - z; ++b)
        for (int m = 0; 2 * m <= d - z; ++m)
          for (int r = 0; r <= m; ++r) n += 2 * r <= d - b - z && 2 * (m - r) <= b;
  return n;
}

template <int P>
__global__ __launch_bounds__(256) void k_upward(const int32_t* __restrict__ list, int nlist, LevelDev lv,
                                                LevelDev lvc, CommonDev cm) {
  constexpr int K = nmi(P);
  constexpr int NE = nmi_entries(P);
  constexpr int CB = upward_cells(P);         // cells per chunk
  __shared__ double sY[CB][8][K];
  __shared__ double sV[CB][K];
  __shared__ double sW[NE];
  __shared__ int sE[NE];
  __shared__ int sB[K + 1];
  __shared__ int sRc[CB][8];
  __shared__ double sM[CB][8];
  constexpr int NF = fold_entries(P);
  __shared__ double sFw[NF];
  __shared__ int16_t sFl[NF], sFs[nh(P) + 1];
  const int t = threadIdx.x;
  for (int i = t; i < NF; i += 256) {
    sFw[i] = cm.fold_w[i];
    sFl[i] = cm.fold_list[i];
  }
  for (int i = t; i <= nh(P); i += 256) sFs[i] = (int16_t)cm.fold_start[i];
  for (int i = t; i < NE; i += 256) {
    sW[i] = cm.m2m_w[i];
    sE[i] = cm.m2m_list[i];
  }
  for (int i = t; i <= K; i += 256) sB[i] = cm.m2m_start[i];
  const int c = t / K, a = t - c * K;
  // children of a chunk: refined rank and mass (the gathered mass of a refined
  // child is 0 and unused), two independent loads, prefetched one chunk ahead
  auto child = [&](int i0, int& rc, double& m) {
    rc = -1;
    m = 0.0;
    const int i = i0 + (t >> 3);
    if (t < CB * 8 && i < nlist) {
      const int ch = 8 * list[i] + (t & 7);
      rc = lvc.rank[ch];
      m = lvc.mass[ch];
    }
  };
  int rcn;
  double mn;
  child(blockIdx.x * CB, rcn, mn);
  for (int i0 = blockIdx.x * CB; i0 < nlist; i0 += gridDim.x * CB) {
    if (t < CB * 8) {
      sRc[t >> 3][t & 7] = rcn;
      sM[t >> 3][t & 7] = rcn < 0 ? mn : 0.0;
    }
    child(i0 + gridDim.x * CB, rcn, mn);
    __syncthreads();
    // a cell whose 8 children are leaves has only monopole children: its signed
    // sums vanish for k > 0 and each coefficient keeps the k = 0 entry (the
    // first of its list)
    auto leaf_only = [&](int cc) {
      bool lo = true;
#pragma unroll
      for (int o = 0; o < 8; ++o) lo = lo && sRc[cc][o] < 0;
      return lo;
    };
    // 8 child values per (cell, coefficient) -> signed sums over the octant bits
    for (int i = t; i < CB * K; i += 256) {
      const int cc = i / K, k = i - cc * K;
      if (k > 0 && leaf_only(cc)) continue;
      double v[8];
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        const int rc = sRc[cc][o];
        v[o] = rc >= 0 ? lvc.S64[(size_t)rc * K + k] : (k == 0 ? sM[cc][o] : 0.0);
      }
#pragma unroll
      for (int bit = 0; bit < 3; ++bit) {
        double u[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int qlo = q & ~(1 << bit);
          u[q] = (q & (1 << bit)) ? v[qlo | (1 << bit)] - v[qlo] : v[qlo] + v[qlo | (1 << bit)];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = u[q];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) sY[cc][q][k] = v[q];
    }
    __syncthreads();
    const int nc = min(CB, nlist - i0);
    if (c < nc) {
      double acc = 0.0;
      if (leaf_only(c)) {
        acc = sW[sB[a]] * sY[c][sE[sB[a]] >> 12][0];
      } else {
        for (int j = sB[a]; j < sB[a + 1]; ++j) {
          const int e = sE[j];
          acc += sW[j] * sY[c][e >> 12][e & 4095];
        }
      }
      lv.S64[(size_t)list[i0 + c] * K + a] = acc;
      sV[c][a] = acc;
    }
    __syncthreads();
    // source copies for the translation kernels carry the factor (-1)^|a|/a! 2^|a|
    store_copies<P>(nc, lv, [&](int cc) { return list[i0 + cc]; }, [&](int cc, int h) {
      double v = 0.0;
      for (int j = sFs[h]; j < sFs[h + 1]; ++j) v += sFw[j] * sV[cc][sFl[j]];
      return v;
    });
    __syncthreads();
  }
}

// Upward pass for the refined cells whose 8 children are leaves (P2M, Eq.
// eq:P2M): the signed child sums vanish for k > 0, so coefficient a is the
// k = 0 entry of its M2M list times one signed sum of the 8 masses (signs by
// the parity of a), and a folded source coefficient, whose terms all have one
// parity, a fixed weight times one such sum.  A block takes kP2mCells cells of
// the list: their masses and the 8 signed sums go to LDS, and the three copies
// (S64 in coefficient order, the scaled FP32 and FP64 copies in their
// layouts) are written slot by slot in row order.
constexpr int kP2mCells = 8;

template <int P>
__global__ __launch_bounds__(256) void k_p2m_leaf(const int32_t* __restrict__ list, int nlist, LevelDev lv,
                                                  LevelDev lvc, CommonDev cm) {
  constexpr int K = nmi(P);
  constexpr int KH = nh(P);
  constexpr int NC = kP2mCells;
  constexpr HTab<P> ht{};
  __shared__ int sR[NC];
  __shared__ double sM[NC][8];
  __shared__ double sY[NC][8];
  __shared__ double sW[K], sWh[KH];
  __shared__ int8_t sQ[K], sQh[KH];
  const int t = threadIdx.x;
  const int c0 = blockIdx.x * NC;
  const int nc = min(NC, nlist - c0);
  if (t < NC) sR[t] = t < nc ? list[c0 + t] : -1;
  if (t < K) {
    const int e0 = cm.m2m_start[t];
    sW[t] = cm.m2m_w[e0];
    sQ[t] = (int8_t)(cm.m2m_list[e0] >> 12);
  }
  __syncthreads();
  if (t < 8 * nc) sM[t >> 3][t & 7] = as_global(lvc.mass)[8 * (size_t)sR[t >> 3] + (t & 7)];
  if (t < KH) {
    sWh[t] = cm.fold_p2m[t];
    sQh[t] = sQ[ht.full[t]];
  }
  __syncthreads();
  if (t < 8 * nc) {
    const int c = t >> 3, q = t & 7;
    double v[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) v[o] = sM[c][o];
    // signed sum over the octant bits of q (the butterfly of k_upward, one output)
#pragma unroll
    for (int bit = 0; bit < 3; ++bit) {
      double u[8];
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        const int lo = o & ~(1 << bit);
        u[o] = (q & (1 << bit)) ? v[lo | (1 << bit)] - v[lo] : v[lo] + v[lo | (1 << bit)];
      }
#pragma unroll
      for (int o = 0; o < 8; ++o) v[o] = u[o];
    }
    sY[c][q] = v[0];
  }
  __syncthreads();
  for (int i = t; i < nc * K; i += 256) {
    const int c = i / K, a = i - c * K;
    lv.S64[(size_t)sR[c] * K + a] = sW[a] * sY[c][sQ[a]];
  }
  store_copies<P>(nc, lv, [&](int c) { return sR[c]; }, [&](int c, int h) { return sWh[h] * sY[c][sQh[h]]; });
}

__global__ void k_batch_in(int64_t nleaf, const int32_t* __restrict__ leafslot, const int32_t* __restrict__ leafhier,
                           const int64_t* __restrict__ base, const double* const* __restrict__ mass,
                           double* __restrict__ m_forest) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nleaf) return;
  const int32_t s = leafslot[i], h = leafhier[i];
  m_forest[s] = mass[h][s - base[h]];
}

__global__ void k_batch_out(int64_t nleaf, const int32_t* __restrict__ leafslot, const int32_t* __restrict__ leafhier,
                            const int64_t* __restrict__ base, const double* __restrict__ phi_forest,
                            const double* __restrict__ acc_forest, double* const* __restrict__ phi,
                            double* const* __restrict__ acc) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nleaf) return;
  const int32_t s = leafslot[i], h = leafhier[i];
  const int64_t j = s - base[h];
  phi[h][j] = phi_forest[s];
  acc[h][3 * j + 0] = acc_forest[3 * (int64_t)s + 0];
  acc[h][3 * j + 1] = acc_forest[3 * (int64_t)s + 1];
  acc[h][3 * j + 2] = acc_forest[3 * (int64_t)s + 2];
}

hipError_t launch_batch_in(int64_t nleaf, const int32_t* leafslot, const int32_t* leafhier, const int64_t* base,
                           const double* const* mass, double* m_forest, hipStream_t st) {
  if (nleaf <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_in, dim3((unsigned)((nleaf + 255) / 256)), dim3(256), 0, st, nleaf, leafslot, leafhier,
                     base, mass, m_forest);
  return hipGetLastError();
}

hipError_t launch_batch_out(int64_t nleaf, const int32_t* leafslot, const int32_t* leafhier, const int64_t* base,
                            const double* phi_forest, const double* acc_forest, double* const* phi,
                            double* const* acc, hipStream_t st) {
  if (nleaf <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_out, dim3((unsigned)((nleaf + 255) / 256)), dim3(256), 0, st, nleaf, leafslot,
                     leafhier, base, phi_forest, acc_forest, phi, acc);
  return hipGetLastError();
}

hipError_t launch_upward(int p, const int32_t* leaf, int nleaf, const int32_t* mix, int nmix, const LevelDev& lv,
                         const LevelDev& lvc, const CommonDev& cm, hipStream_t st) {
  const int CB = upward_cells(p);
  if (nleaf > 0) {
    const dim3 grid((unsigned)((nleaf + kP2mCells - 1) / kP2mCells)), block(256);
    switch (p) {
#define AFMM_P2M(PP) \
  case PP: hipLaunchKernelGGL(k_p2m_leaf<PP>, grid, block, 0, st, leaf, nleaf, lv, lvc, cm); break;
      AFMM_P2M(1) AFMM_P2M(2) AFMM_P2M(3) AFMM_P2M(4) AFMM_P2M(5) AFMM_P2M(6) AFMM_P2M(7) AFMM_P2M(8)
#undef AFMM_P2M
      default: return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (nmix > 0) {
    // persistent blocks: a few per CU, each looping over chunks of CB cells
    const dim3 grid(std::min((nmix + CB - 1) / CB, 8 * 256)), block(kBlock);
    switch (p) {
#define AFMM_UP(PP) \
  case PP: hipLaunchKernelGGL(k_upward<PP>, grid, block, 0, st, mix, nmix, lv, lvc, cm); break;
      AFMM_UP(1) AFMM_UP(2) AFMM_UP(3) AFMM_UP(4) AFMM_UP(5) AFMM_UP(6) AFMM_UP(7) AFMM_UP(8)
#undef AFMM_UP
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Completion of the local expansions of FMM level f (one block per M2L group
// F): the M2L sums of the KH coefficients with c <= 1 (split over `nsplit`
// tap ranges, added in fixed order; or the single sum at the front of the row
// of L), the coefficients with c >= 2 that follow from them (harmonic
// relation), and the ShiftLocal term sum_g w_o[|b|][g] L~_{b+g}[F] (Eq. eq:L2L)
// when F has one.  Three passes over the group's coefficients through LDS: the
// tap sums and the stores run coefficient-fastest (whole child rows per wave),
// the expansion and shift sums child-fastest.  NS bounds the split (1: the
// single sum in L): every partial of every coefficient a thread owns is loaded
// at once, so a block waits for one round of loads rather than one per four
// partials and coefficient.
template <typename T, typename TL, int P, int NS>
__global__ __launch_bounds__(kBlock) void k_l2l(const int32_t* __restrict__ grp, const TL* __restrict__ Lpar,
                                                const int32_t* __restrict__ rank0, T* __restrict__ Lout,
                                                const T* __restrict__ Lpart, int nsplit, size_t split_stride,
                                                const T* __restrict__ w, const int16_t* __restrict__ sumidx,
                                                const int8_t* __restrict__ mi) {
  constexpr int K = nmi(P), KH = nh(P);
  constexpr int KV = K | 1, KHV = KH | 1;  // odd LDS row strides: the 8 rows of a wave's accesses fall in different banks
  __shared__ T sL[K];
  __shared__ T sH[8 * KHV];
  __shared__ T sV[8 * KV];
  __shared__ int sRy[8];
  const int F = grp[blockIdx.x];
  const int t = threadIdx.x;
  if (t < K && Lpar) sL[t] = (T)Lpar[(size_t)F * K + t];
  if (t < 8) sRy[t] = rank0[8 * F + t];
  __syncthreads();
  // tap sums, coefficient fastest (each child's row is read contiguously);
  // a thread owns coefficients t, t + 256, ... (NI of them); a missing child
  // row reads row 0 and is not stored
  constexpr int NI = (8 * KH + kBlock - 1) / kBlock;
  {
    T x[NI][NS];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int i = min(t + kBlock * j, 8 * KH - 1), o = i / KH, b = i - o * KH;
      const int ry = sRy[o];
      const size_t at = (size_t)(ry >= 0 ? ry : 0) * (NS == 1 ? K : KH) + b;
#pragma unroll
      for (int c = 0; c < NS; ++c) x[j][c] = NS == 1 ? Lout[at] : Lpart[min(c, nsplit - 1) * split_stride + at];
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int i = t + kBlock * j;
      if (i >= 8 * KH) break;
      const int o = i / KH, b = i - o * KH;
      if (sRy[o] < 0) continue;
      T v = 0;
      if constexpr (NS == 1) {
        v = x[j][0];
      } else {
#pragma unroll
        for (int c = 0; c < NS; ++c)
          if (c < nsplit) v += x[j][c];
      }
      sH[o * KHV + b] = v;
    }
  }
  __syncthreads();
  // coefficient (i, j, k + 2m), k <= 1, is (-1)^m sum_r C(m, r) of (i + 2r, j +
  // 2(m - r), k); then ShiftLocal.  Child o fastest: the lanes of a wave share few
  // coefficients b, all of nearly the same degree, so their sums have nearly
  // equal lengths
  for (int i = t; i < 8 * K; i += kBlock) {
    const int o = i & 7, b = i >> 3;
    if (sRy[o] < 0) continue;
    const int nb = mi[4 * b + 3], m = mi[4 * b + 2] >> 1;
    const T* h = sH + o * KHV + nb * nb + (mi[4 * b + 2] & 1) * (nb + 1) + mi[4 * b + 1] + 2 * m;
    T v = h[0];
    for (int r = 1, c = m; r <= m; ++r) {
      v += (T)c * h[-2 * r];
      c = c * (m - r) / (r + 1);
    }
    if (m & 1) v = -v;
    if (Lpar) {
      const T* wr = w + ((size_t)o * (P + 1) + nb) * K;
      const int16_t* si = sumidx + (size_t)b * K;
      T sh = 0;
      for (int g = 0; g < nmi(P - nb); ++g) sh += wr[g] * sL[si[g]];
      v += sh;
    }
    sV[o * KV + b] = v;
  }
  __syncthreads();
  for (int i = t; i < 8 * K; i += kBlock) {
    const int o = i / K, b = i - o * K;
    const int ry = sRy[o];
    if (ry >= 0) Lout[(size_t)ry * K + b] = sV[o * KV + b];
  }
}

// ---------------------------------------------------------------------------
// Tap pipeline of M2L up to p = 4.  A block owns 16 groups of one parity class at one
// level.  For each of the 189 taps:
//   sB[k][n] = folded coefficient k of the tap's source of group n (its mass for
//             a leaf source, 0 when there is none): thread (n, q) loads block q
//             of the source row and stores its values by coefficient;
//   sD[o][g] = D~_g at the tap's child offset o (8 rows, then one zero slot)
//             is staged in LDS while the MFMAs of the previous tap run.
// A fragments are read from sD through per-lane offsets that do not depend on
// the tap (kept in registers).
// The first k-step (monopole and dipole terms, by far the largest) and the
// others sum into separate accumulators in the lowest rows: folded, the terms
// of orders >= 2 no longer come as large values of opposite sign, and many are
// below half a unit in the last place of the running sum; in one FP32
// accumulator they were rounded away on one side (the potential's mean error
// rose from 0.4e-7 to 7e-7 at p = 6).
template <typename T, int P>
struct TapStage {
  static constexpr int K = nh(P);            // folded coefficients
  static constexpr int KP = (K + 3) & ~3;    // coefficients covered by the k-steps
  static constexpr int KS = dstage_ks(P);    // sD row stride
  static constexpr int VW = 16 / (int)sizeof(T);
  static constexpr int ROW = src_row(P, (int)sizeof(T));  // source-copy row length
  static constexpr int SD = 8 * KS + 1;      // sD size (8 rows + zero slot)
  static constexpr int SDP = dstage_len(P, (int)sizeof(T));  // staged length (16-byte padded)
  static constexpr int NDV = SDP / VW;       // 16-byte vectors of one stage
  static constexpr int SB = 16 * KP + 16;    // sB size (k-steps, then a row for the unused slots)
};

// scaled source copies c_a 2^|a| S~_a of a level
template <typename T> __device__ inline const T* level_S(const LevelDev& lv);
template <> __device__ inline const float* level_S<float>(const LevelDev& lv) { return lv.S32; }
template <> __device__ inline const double* level_S<double>(const LevelDev& lv) { return lv.Sc64; }
template <typename T> __device__ inline T* level_L(const LevelDev& lv);
template <> __device__ inline float* level_L<float>(const LevelDev& lv) { return lv.L32; }
template <> __device__ inline double* level_L<double>(const LevelDev& lv) { return lv.L64; }

// Drops the taps of a range that have no source in any of the 16 columns
// (they add nothing; common near the box faces), keeping the order: run by
// one whole wave, in place on the source table src[tap][16], with the taps'
// codes copied to code[].  Returns the number kept (at least 1: an empty
// range keeps its first tap, whose B is zero).
__device__ inline int compact_taps(int nt, const int32_t* __restrict__ tp, int* src, int* code) {
  const int lane = threadIdx.x & 63;
  int cnt = 0;
  for (int i0 = 0; i0 < nt; i0 += 64) {
    const int i = i0 + lane;
    int v[16];
    bool any = false;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      v[c] = i < nt ? src[i * 16 + c] : -1;
      any = any || v[c] != -1;
    }
    const int cd = i < nt ? tp[i] : 0;
    const uint64_t m = __ballot(any);
    wave_sync();
    if (any) {
      const int j = cnt + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
      for (int c = 0; c < 16; ++c) src[j * 16 + c] = v[c];
      code[j] = cd;
    }
    cnt += __popcll(m);
    wave_sync();
  }
  if (cnt == 0) {
    if (lane < 16) src[lane] = -1;
    if (lane == 0) code[0] = tp[0];
    cnt = 1;
  }
  wave_sync();
  return cnt;
}

// Tap range of chunk c of nsplit: whole pairs of taps (the tap loops run in
// pairs), so that only the last chunk has an odd count and runs one empty tap.
// The host keeps nsplit <= 21, so every range holds at least 8 taps.
__host__ __device__ inline void tap_range(int c, int nsplit, int& tb, int& te) {
  constexpr int kPairs = (kTaps + 1) / 2;
  tb = 2 * (c * kPairs / nsplit);
  te = min(kTaps, 2 * ((c + 1) * kPairs / nsplit));
}

// Source of column n for tap `code`: refined rank (>= 0), -2 - cell for a leaf
// (monopole), or -1 when there is none.  The tap loops resolve the sources of
// all their taps into LDS before the loop.
__device__ inline int tap_src(int code, int n, const int* __restrict__ sCB, gptr<int32_t> rank1) {
  const int cb = sCB[n * 27 + (code & 31)];
  const int s = cb < 0 ? -1 : cb + ((code >> 5) & 7);
  if (s < 0) return -1;
  const int rs = rank1[s];
  return rs >= 0 ? rs : -2 - s;
}

template <typename T, int P, int NTH>
__device__ inline void store_dstage(T* sD, const typename Vec16<T>::type* vD) {
  using TS = TapStage<T, P>;
  using V = typename Vec16<T>::type;
  constexpr int NJ = (TS::NDV + NTH - 1) / NTH;
  const int t = threadIdx.x;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (TS::NDV % NTH == 0 || t + NTH * j < TS::NDV) ((V*)sD)[t + NTH * j] = vD[j];
}

// Block-local setup: the tile record (level, then NC groups) and, per group,
// the child base (8 x refined rank) of each of its father's 27 neighbours.
__device__ inline void tile_setup(const int32_t* __restrict__ rec, int NC, const LevelDev& lv2,
                                  const LevelDev& lv1, int* sF, int* sCB) {
  const int t = threadIdx.x;
  if (t < NC) sF[t] = rec[1 + t];
  __syncthreads();
  for (int i = t; i < NC * 27; i += kBlock) {
    const int n = i / 27, e = i - n * 27;
    const int F = sF[n];
    int v = -1;
    if (F >= 0) {
      const int G = as_global(lv1.refcell)[F] >> 3;
      const int Q = as_global(lv2.nbr)[(size_t)G * 27 + e];
      if (Q >= 0) {
        const int rQ = as_global(lv2.rank)[Q];
        if (rQ >= 0) v = 8 * rQ;
      }
    }
    sCB[i] = v;
  }
}


// ---------------------------------------------------------------------------
// Intermediate-field M2P at the leaves (Alg. 4 / Sec. 3.2), by the reflections of
// the axes.  Reflecting an axis maps a source offset d onto another, the child
// offsets onto each other, and D~_g onto (-1)^(g_i) D~_g; so over an orbit of
// offsets (afmm_internal.h) the map from the sources' coefficients to the
// children's values splits by the 8 characters chi of the reflections:
//   U_chi[a]  = sum over the orbit's sources of chi(sigma) sigma^a S_sigma[a]
//   V_chi,i   = sum_a A_chi,i[a] U_chi[a]      i = phi, ax, ay, az
//   value_i(o) = tau_i sum_chi chi(tau) V_chi,i,   tau = the signs of child o
// with A_chi,i[a] = E_(chi ^ e_i)[a + e_i], E the characters of the D~ rows.  An
// orbit of 1, 2, 4 or 8 sources costs 8 x 4 x KH products, as much as one source
// in the direct form: 56 orbits instead of 189 taps.
//
// A block takes up to 48 or 64 groups of one parity class (12 or 16 per wave) and
// a range of the orbits.  The sources of the 7 orbits of one m sit in one octant of
// their fathers, so the rows of that octant of all fathers of the tile (their
// number is bounded by the tile) are staged in LDS once and read from there about
// six times; read from memory for each use they were 50 GB at 8M leaves (now the
// L2s give 24 GB, half of it operators).  The distinct fathers are found through a hash
// table in LDS.
// 4x4 blocks of MFMA: lane (q = lane >> 2, j = lane & 3) holds the coefficients of
// block q (SymLayout) of group j of a quad; all coefficients of a block have one
// parity, so sigma^a is one sign per lane and axis, and the sources' vectors turn
// into the U_chi by butterflies in registers.  One MFMA takes element e of every
// block for one chi (FP32: 16 blocks of 4 x 4 x 1, the blocks summed at the end;
// FP64: 4 blocks of 4 x 4 x 4).  The A operand of an orbit (32 values a lane and
// pass) comes through a ring of three steps in LDS, shared by the block, and stays
// in registers for the wave's quads.  Output: part[F][i * 8 + o] (accelerations
// negated), one partial set per orbit range.
// Matrix and vector instructions of one SIMD do not overlap here (32 of each take
// their sum one after the other, more interleaved), and at two waves per SIMD the butterflies, the LDS
// reads behind them and the MFMAs share the time about evenly.  8.08M leaves
// (128^3 + 4 levels) at p = 6 FP32: 8.7 ms summed tap by tap over all K
// coefficients, 6.4 on the folded ones, 4.95 by orbits; 287,680 leaves FP64: 703,
// 501, 368 us; 64^3 and 128^3 batches at p = 4 and 8 FP32: 1494 to 866, 1903 to 986.
//
// Groups far apart fill a tile's fathers long before its columns.  They go to direct
// tiles (STAGED false; the host's rule is at append_m2p_tiles): the row and the mass of
// every (neighbour, column) are resolved once per octant of m, the next octant's while
// this one runs, and the sources' rows come from memory, a quad or the first quad
// of the next orbit ahead.  Same sums in the same order, so the same bits.  They are
// bound by the latency of those loads and share k_m2p, for one launch covers the tiles
// of all levels; the registers of both forms decide the occupancy (FP64 to p = 3 runs
// three blocks per CU, which the loads of the next octant's sources would exceed).
// Finest level of 64^3 + 2% of its cells (5243 groups), staged / direct: 93 / 63 us at
// p = 3 FP64, 110 / 65 at p = 4, 182 / 64 at p = 6 FP32, 316 / 104 at p = 6 FP64; tap
// by tap, 16 groups per tile wherever they lie, they took 64, 57, 90 and 143.
template <typename T> struct M2PAcc { typedef f32x4 type; };
template <> struct M2PAcc<double> { typedef double type; };
__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0); }
__device__ inline double mfma4(double a, double b, double c) { return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0); }

template <typename T, int P, bool STAGED>
struct M2P {
  using SL = SymLayout<P, (int)sizeof(T)>;
  static constexpr int CP = SL::CP, NP = SL::NP, ROW = SL::ROW;
  static constexpr int NQ = m2p_quads(P, (int)sizeof(T)), COLS = m2p_cols(P, (int)sizeof(T));
  static constexpr int NF = m2p_fathers(P, (int)sizeof(T)), LV = m2p_vec(P, (int)sizeof(T));
  static constexpr int AL = 8 * 64 * CP;    // A values of one orbit and pass
  static constexpr int NH = 512;            // hash slots
  static_assert(NF <= kBlock && 2 * NF <= NH, "one father per thread, table half full");
  typedef typename VecN<T, CP>::type V;
  typedef typename M2PAcc<T>::type Acc;
  struct Hash {
    int key[NH];
    uint16_t slot[NH];
  };
  struct LdsStaged {
    union {
      T rows[(NF + 1) * kSymBlocks * LV];   // the octant's rows (block q of row u at place q ^ (u & 15)), then zeros
      Hash h;
    };
    T a[3][AL];                             // ring over steps (m, pass, orbit)
    int src[2][NF];                         // sources of the octant (and of the next one): rank, or -2 - cell
    int base[NF];                           // children of the distinct fathers
    uint16_t tab[27 * COLS];                // row of neighbour e of column n's father, as the byte place of its block 0
    int F[COLS];
    int wsum[4];
    int nf;
  };
  struct LdsDirect {
    T a[3][AL];
    int base[27 * COLS];                    // children of neighbour e of column n's father, or -1
    int row[27 * COLS];                     // row of the one in the octant (the zero row for a leaf or none)
    T mass[27 * COLS];                      // its mass if it is a leaf, else 0
    int F[COLS];
  };
  using Lds = std::conditional_t<STAGED, LdsStaged, LdsDirect>;
  Lds& l;
  const T* __restrict__ symA;
  const uint64_t* __restrict__ taps;        // fathers of the class's orbits, a byte each
  gptr<int32_t> rank1;
  gptr<double> mass1;
  gptr<T> S;                                // the level's source copy
  int zrow, nf, C, par;
  int nq;                                   // quads of a wave that hold groups (not STAGED)
  int ps;                                   // pass of the steps that run (not STAGED)
  int g0, g1;                               // steps (m, pass, j) of this block: [g0, g1) of 56 NP
  int af;                                   // axes on which the operand being loaded has its far offset on the other side
  int ra, wa;                               // ring places: operand of the next step, of the one after
  T sg[3];                                  // sigma^a sign of this lane's block on each axis
  Acc acc[NQ][8];
  V a[8], an[2], first[STAGED ? 1 : 8];

  static constexpr int axis(int pt, int b) {  // b-th axis of the set
    int i = 0;
    for (; i < 3; ++i)
      if (pt >> i & 1 && b-- == 0) break;
    return i;
  }
  static constexpr int sub(int pt, int chi) {  // chi restricted to the set, as an index over its axes
    int r = 0, b = 0;
    for (int i = 0; i < 3; ++i)
      if (pt >> i & 1) r |= (chi >> i & 1) << b++;
    return r;
  }
  // The lane, opaque: the addresses that follow from it are formed where they are
  // used; hoisted out of the step loop, dozens of them went to scratch, and their
  // reloads waited for every load in flight.
  static __device__ inline int lane_id() {
    int x = threadIdx.x & 63;
    asm volatile("" : "+v"(x));
    return x;
  }
  static __device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

  // byte place in LDS of block q of row u; block q of the row at place p is at p ^ place(0, q)
  static constexpr int VB = LV * (int)sizeof(T);
  static_assert((NF + 1) * kSymBlocks * VB <= 65536, "places fit 16 bits");
  static __device__ inline int place(int u, int q) { return (u * kSymBlocks + (q ^ (u & 15))) * VB; }

  // The distinct refined fathers among the neighbours of the columns' fathers:
  // every (column, neighbour) enters its rank into the table, the occupied slots
  // are numbered, and tab takes the numbers (NF, the zero row, for none).
  __device__ inline void find_fathers(gptr<int32_t> refcell1, gptr<int32_t> nbr2, gptr<int32_t> rank2) {
    const int t = threadIdx.x;
    constexpr int NE = (27 * COLS + kBlock - 1) / kBlock;
    int key[NE], at[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int i = t + kBlock * k, e = i / COLS, F = i < 27 * COLS ? l.F[i - e * COLS] : -1;
      const int Q = F >= 0 ? nbr2[(size_t)(refcell1[F] >> 3) * 27 + e] : -1;
      key[k] = Q >= 0 ? rank2[Q] : -1;
    }
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      at[k] = -1;
      if (key[k] < 0) continue;
      uint32_t h = ((uint32_t)key[k] * 2654435761u) >> 23;  // top 9 bits
      for (int tries = 0; tries < NH; ++tries, h = (h + 1) & (NH - 1)) {
        const int old = atomicCAS(&l.h.key[h], -1, key[k]);
        if (old == -1 || old == key[k]) {
          at[k] = (int)h;
          break;
        }
      }
    }
    __syncthreads();
    const int k0 = l.h.key[2 * t], k1 = l.h.key[2 * t + 1], lane = t & 63;
    const uint64_t m0 = __ballot(k0 >= 0), m1 = __ballot(k1 >= 0), below = (1ull << lane) - 1ull;
    if (lane == 0) l.wsum[t >> 6] = __popcll(m0) + __popcll(m1);
    __syncthreads();
    int b = __popcll(m0 & below) + __popcll(m1 & below);
    for (int v = 0; v < (t >> 6); ++v) b += l.wsum[v];
    if (k0 >= 0 && b < NF) {
      l.h.slot[2 * t] = (uint16_t)b;
      l.base[b++] = 8 * k0;
    }
    if (k1 >= 0 && b < NF) {
      l.h.slot[2 * t + 1] = (uint16_t)b;
      l.base[b++] = 8 * k1;
    }
    if (t == kBlock - 1) l.nf = min(b, NF);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NE; ++k)
      if (t + kBlock * k < 27 * COLS) l.tab[t + kBlock * k] = (uint16_t)place(at[k] >= 0 ? l.h.slot[at[k]] : NF, 0);
    __syncthreads();
  }

  // source of father t in the octant of m
  __device__ inline int source_cell(int m) const {
    return (int)threadIdx.x < nf ? l.base[threadIdx.x] + (C ^ m) : 0;
  }
  __device__ inline void put_source(int m, int cell, int rk) {
    if ((int)threadIdx.x < nf) l.src[m & 1][threadIdx.x] = rk >= 0 ? rk : -2 - cell;
  }
  // rows of the octant of m, pass s; on the last pass, the sources of m + 1
  __device__ inline void stage(int m, int s) {
    const int t = threadIdx.x, q = t & 15;
    const int cell = source_cell(min(m + 1, 7));
    const int rk = rank1[cell];
    constexpr int U = 4;
    for (int u0 = t >> 4; u0 < nf; u0 += 16 * U) {
      V v[U];
      double mm[U];
      int code[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int u = min(u0 + 16 * k, nf - 1);
        code[k] = l.src[m & 1][u];
        v[k] = load_vec<T, CP>(S + (size_t)(code[k] >= 0 ? code[k] : zrow) * ROW + (s * kSymBlocks + q) * CP);
        mm[k] = mass1[code[k] <= -2 ? -2 - code[k] : 0];
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int u = min(u0 + 16 * k, nf - 1);
        if (s == 0 && q == 0 && code[k] <= -2) v[k][0] = (T)mm[k];  // a leaf: its mass
        store_vec<T, CP>((T*)((char*)l.rows + place(u, q)), v[k]);
      }
    }
    if (s == NP - 1 && m + 1 < 8) put_source(m + 1, cell, rk);
    __syncthreads();
  }
  // not STAGED: children of the neighbours of the columns' fathers
  __device__ inline void find_bases(gptr<int32_t> refcell1, gptr<int32_t> nbr2, gptr<int32_t> rank2) {
    for (int i = threadIdx.x; i < 27 * COLS; i += kBlock) {
      const int e = i / COLS, F = l.F[i - e * COLS];
      const int Q = F >= 0 ? nbr2[(size_t)(refcell1[F] >> 3) * 27 + e] : -1, r = Q >= 0 ? rank2[Q] : -1;
      l.base[i] = r >= 0 ? 8 * r : -1;
    }
    __syncthreads();
  }
  // not STAGED: the sources in the octant of m on their way, and into LDS.  The
  // masses of refined cells are 0 and so are the values of the zero row, so a
  // source is its row plus its mass.
  static constexpr int NE = (27 * COLS + kBlock - 1) / kBlock;
  static constexpr bool AHEAD = sizeof(T) == 4 || P > 3;  // registers
  struct Sources {
    int rk[NE];
    double mm[NE];
  };
  __device__ inline void load_sources(int m, Sources& r) const {
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int b = l.base[min((int)threadIdx.x + kBlock * k, 27 * COLS - 1)];
      r.rk[k] = -1;
      r.mm[k] = 0.0;
      if (b >= 0) {
        r.rk[k] = rank1[b + (C ^ m)];
        r.mm[k] = mass1[b + (C ^ m)];
      }
    }
  }
  __device__ inline void put_sources(const Sources& r) {
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int i = threadIdx.x + kBlock * k;
      if (i >= 27 * COLS) continue;
      l.row[i] = r.rk[k] >= 0 ? r.rk[k] : zrow;
      l.mass[i] = (T)r.mm[k];
    }
    __syncthreads();
  }
  // the block's share of the A operand of step g (the last one past the end):
  // characters wave, wave + 4; put into the ring with the sign of this class: the
  // operator's representative offsets are positive, mirrored on the axes on which
  // the class has its far offset on the other side
  __device__ inline void load_a(int g) {
    const int lane = lane_id(), wv = wave_id();
    g = min(g, g1 - 1);
    const int ms = g / 7, m = ms / NP;
    af = C & m & ~sym_axes(sym_set(m, g - 7 * ms));
    gptr<T> src = as_global(symA + ((size_t)g * AL + wv * 64 * CP)) + lane * CP;
#pragma unroll
    for (int r = 0; r < 2; ++r) an[r] = load_vec<T, CP>(src + 4 * 64 * CP * r);
  }
  __device__ inline void put_a(int place) {
    const int lane = lane_id(), wv = wave_id();
    if (af) {
#pragma unroll
      for (int r = 0; r < 2; ++r) an[r] *= __popc((par ^ (wv + 4 * r)) & af) & 1 ? (T)-1 : (T)1;
    }
    T* ring = l.a[place] + (wv * 64 + lane) * CP;
#pragma unroll
    for (int r = 0; r < 2; ++r) store_vec<T, CP>(ring + 4 * 64 * CP * r, an[r]);
  }
  __device__ inline void read_a(int c, int lane, int place) {
    a[c] = load_vec<T, CP>((const T*)l.a[place] + (c * 64 + lane) * CP);
  }
  template <int PT>
  __device__ inline void transform(V* v) const {
    constexpr int NB = sym_bits(PT);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const T s = sg[axis(PT, b)];
#pragma unroll
      for (int i = 0; i < 1 << NB; ++i)
        if (!(i >> b & 1)) {
          const V p = v[i], m = v[i | 1 << b];
#pragma unroll
          for (int e = 0; e < CP; ++e) {
            v[i][e] = p[e] + s * m[e];
            v[i | 1 << b][e] = p[e] - s * m[e];
          }
        }
    }
  }
  // row of source i of an orbit (its fathers in code) for quad qd of the wave: block q
  __device__ inline V source_row(uint64_t code, int i, int qd, int lane) const {
    const int at = ((int)(code >> (8 * i)) & 31) * COLS + (wave_id() * NQ + qd) * 4 + (lane & 3);
    if constexpr (STAGED) return load_vec<T, CP>((const T*)((const char*)l.rows + (l.tab[at] ^ (lane >> 2) * VB)));
    else return load_vec<T, CP>(S + (size_t)l.row[at] * ROW + (ps * kSymBlocks + (lane >> 2)) * CP);
  }
  // not STAGED: the first quad's rows of the next orbit, of at most N sources (bytes of
  // code past the orbit's sources are 0, a valid neighbour), on their way
  template <int N>
  __device__ inline void load_first(uint64_t code, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) first[i] = source_row(code, i, 0, lane);
  }
  // one orbit and pass: the wave's quads.  Butterflies and products apart: these MFMAs
  // and the VALU share the units, and every change between them costs some cycles
  // (32 of each: 541 cycles interleaved, 421 one after the other, two waves).  One
  // quad's reads ahead, no more (registers).
  template <int PT, int NEXT>
  __device__ inline void orbit(uint64_t code, uint64_t next) {
    constexpr int NS = 1 << sym_bits(PT);
    const int lane = lane_id();
    auto products = [&](int qd, V* v) {
      transform<PT>(v);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < CP; ++e)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[qd][c] = mfma4(a[c][e], v[sub(PT, c)][e], acc[qd][c]);
    };
    if constexpr (STAGED) {
      V v[2][NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) v[0][i] = source_row(code, i, 0, lane);
#pragma unroll
      for (int qd = 0; qd < NQ; ++qd) {
        if (qd + 1 < NQ)
#pragma unroll
          for (int i = 0; i < NS; ++i) v[(qd + 1) & 1][i] = source_row(code, i, qd + 1, lane);
        products(qd, v[qd & 1]);
        if (qd == NQ - 1)
#pragma unroll
          for (int c = 0; c < 8; ++c) read_a(c, lane, ra);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      V odd[NS];
#pragma unroll
      for (int qd = 0; qd < NQ; ++qd) {
        if (qd >= nq) break;
        V *v = qd & 1 ? odd : first, *ahead = qd & 1 ? first : odd;
        if (qd + 1 < NQ && qd + 1 < nq)
#pragma unroll
          for (int i = 0; i < NS; ++i) ahead[i] = source_row(code, i, qd + 1, lane);
        if (ps == 0) {
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            const T mm = l.mass[((int)(code >> (8 * i)) & 31) * COLS + (wave_id() * NQ + qd) * 4 + (lane & 3)];
            v[i][0] += lane < 4 ? mm : (T)0;
          }
        }
        products(qd, v);
        __builtin_amdgcn_sched_barrier(0);
      }
      load_first<NEXT>(next, lane);
#pragma unroll
      for (int c = 0; c < 8; ++c) read_a(c, lane, ra);
    }
  }
  __device__ inline uint64_t sources_of(int g) const {
    g = min(g, g1 - 1);
    return taps[g / (7 * NP) * 7 + g % 7];
  }
  // the steps of one phase, h the step of the TY-th set: one after the other
  // (behind a switch the accumulators were copied)
  template <int TY>
  __device__ inline void sets(int m, int h, int& g, uint64_t& code) {
    const bool on = sym_axes(TY) != m;
    if (on && h == g && g < g1) {
      const uint64_t c = code;
      code = sources_of(g + 1);
      put_a(wa);
      load_a(g + 3);
      orbit<sym_axes(TY), 1 << sym_bits(sym_axes(TY < 7 ? TY + 1 : 7))>(c, code);
      const int x = 3 - ra - wa;  // the place of the operand just used
      ra = wa;
      wa = x;
      ++g;
      __syncthreads();
    }
    if constexpr (TY < 7) sets<TY + 1>(m, on ? h + 1 : h, g, code);
  }
  __device__ inline void run() {
    int g = g0;
    uint64_t code = sources_of(g);
    std::conditional_t<STAGED, char, Sources> next;
    if constexpr (!STAGED && AHEAD) load_sources(g0 / (7 * NP), next);
    while (g < g1) {
      const int ms = g / 7, m = ms / NP;
      if constexpr (STAGED) {
        stage(m, ms - m * NP);
      } else {
        ps = ms - m * NP;
        if (ps == 0 || g == g0) {
          if (!AHEAD) load_sources(m, next);
          put_sources(next);
          if (AHEAD) load_sources(min(m + 1, 7), next);
        }
        load_first<8>(code, lane_id());
      }
      sets<0>(m, 7 * ms, g, code);
    }
  }
};

// One tile (record rec: the target level, the quads per wave << 8 or 0 for a STAGED
// tile, the groups) and one of nsplit ranges of the orbits.
template <typename T, int P, bool STAGED>
__device__ inline void m2p_tile(typename M2P<T, P, STAGED>::Lds& lds, const int32_t* __restrict__ rec, int chunk, int nsplit,
                                const int8_t* __restrict__ taps, const LevelDev* __restrict__ lvs,
                                const T* __restrict__ symA) {
  using MP = M2P<T, P, STAGED>;
  using SL = typename MP::SL;
  static constexpr SL sl{};
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, q = lane >> 2, j = lane & 3;
  const int level = rec[0] & 255;
  const LevelDev lv1 = lvs[level - 1];
  const LevelDev lv2 = lvs[level - 2];
  if (t < MP::COLS) lds.F[t] = rec[1 + t];
  if constexpr (STAGED) lds.h.key[t] = lds.h.key[t + kBlock] = -1;
  static_assert(MP::NH == 2 * kBlock, "two hash slots per thread");
  __syncthreads();
  gptr<int32_t> refcell1 = as_global(lv1.refcell);
  MP m{lds, symA};
  m.C = __builtin_amdgcn_readfirstlane(refcell1[lds.F[0]] & 7);
  m.taps = (const uint64_t*)taps + m.C * kSymOrbits;
  m.g0 = chunk * (kSymOrbits * MP::NP) / nsplit;
  m.g1 = (chunk + 1) * (kSymOrbits * MP::NP) / nsplit;
  m.S = as_global(level_S<T>(lv1));
  m.rank1 = as_global(lv1.rank);
  m.mass1 = as_global(lv1.mass);
  m.zrow = lv1.nref;
  m.par = sl.par[q];
#pragma unroll
  for (int i = 0; i < 3; ++i) m.sg[i] = m.par >> i & 1 ? (T)-1 : (T)1;
#pragma unroll
  for (int d = 0; d < MP::NQ; ++d)
#pragma unroll
    for (int c = 0; c < 8; ++c) m.acc[d][c] = typename MP::Acc{};
  // the A operand of the first two steps into the ring, the third on its way; the
  // first octant's sources; the zero row
  if constexpr (STAGED) {
    m.find_fathers(refcell1, as_global(lv2.nbr), as_global(lv2.rank));
    m.nf = lds.nf;
    const int mf = m.g0 / (7 * MP::NP), cell = m.source_cell(mf);
    m.put_source(mf, cell, m.rank1[cell]);
    if (t < kSymBlocks * MP::LV) lds.rows[MP::NF * kSymBlocks * MP::LV + t] = 0;
  } else {
    m.nq = rec[0] >> 8;
    m.find_bases(refcell1, as_global(lv2.nbr), as_global(lv2.rank));
  }
  m.load_a(m.g0);
  m.put_a(0);
  m.load_a(m.g0 + 1);
  m.put_a(1);
  m.load_a(m.g0 + 2);
  m.ra = 1;
  m.wa = 2;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 8; ++c) m.read_a(c, lane, 0);
  m.run();
  // characters -> children (index y = ~o), in registers; then the sum over the
  // blocks of coefficients: halves exchanged until each lane holds two values
  gmut<T> part = as_global_mut((T*)lv1.part) + (size_t)chunk * lv1.nref * 32;
#pragma unroll
  for (int d = 0; d < MP::NQ; ++d) {
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (!(c & bit)) {
          const auto x = m.acc[d][c], y = m.acc[d][c | bit];
          m.acc[d][c] = x + y;
          m.acc[d][c | bit] = x - y;
        }
    const int F = lds.F[(wv * MP::NQ + d) * 4 + j];
    if constexpr (sizeof(T) == 4) {
      T v[32];  // i * 8 + o
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int o = 0; o < 8; ++o) {
          const T x = m.acc[d][7 - o][i];
          v[i * 8 + o] = i > 0 && (o >> (i > 0 ? i - 1 : 0) & 1) ? -x : x;
        }
#pragma unroll
      for (int n = 16, lb = 32; n >= 2; n >>= 1, lb >>= 1) {
        const bool up = lane & lb;
#pragma unroll
        for (int k = 0; k < n; ++k) {
          const T keep = up ? v[n + k] : v[k], give = up ? v[k] : v[n + k];
          v[k] = keep + __shfl_xor(give, lb, 64);
        }
      }
      if (F >= 0) {
        gmut<T> out = part + (size_t)F * 32 + 2 * q;
        out[0] = v[0];
        out[1] = v[1];
      }
    } else {
      // lane (i = lane >> 4, block = (lane >> 2) & 3, group j)
      const int i = lane >> 4;
      T v[8];
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        const T x = m.acc[d][7 - o];
        v[o] = i > 0 && (o >> (i - 1) & 1) ? -x : x;
      }
#pragma unroll
      for (int n = 4, lb = 8; n >= 2; n >>= 1, lb >>= 1) {
        const bool up = lane & lb;
#pragma unroll
        for (int k = 0; k < n; ++k) {
          const T keep = up ? v[n + k] : v[k], give = up ? v[k] : v[n + k];
          v[k] = keep + __shfl_xor(give, lb, 64);
        }
      }
      if (F >= 0) {
        gmut<T> out = part + (size_t)F * 32 + i * 8 + 2 * (q & 3);
        out[0] = v[0];
        out[1] = v[1];
      }
    }
  }
}

template <typename T, int P>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(M2P<T, P, false>::AHEAD ? 2 : 3)))
void k_m2p(const int32_t* __restrict__ tiles, int ntiles, int nsplit, const int8_t* __restrict__ taps,
           const LevelDev* __restrict__ lvs, const T* __restrict__ symA) {
  __shared__ __align__(16) union {
    typename M2P<T, P, true>::Lds staged;
    typename M2P<T, P, false>::Lds direct;
  } lds;
  const int item = xcd_tile(ntiles * nsplit);
  if (item >= ntiles * nsplit) return;
  const int tile = item / nsplit, chunk = item - tile * nsplit;
  const int32_t* rec = tiles + (size_t)tile * (m2p_cols(P, (int)sizeof(T)) + 1);
  if (rec[0] < 256) m2p_tile<T, P, true>(lds.staged, rec, chunk, nsplit, taps, lvs, symA);
  else m2p_tile<T, P, false>(lds.direct, rec, chunk, nsplit, taps, lvs, symA);
}

// ---------------------------------------------------------------------------
// M2L tap sums up to p = 4 (Alg. 3 without the ShiftLocal term, which
// the L2L chain adds afterwards): rows R = 8 b + o (local coefficient b, child
// octant o; b in degree order, so 16-row tile T starts at coefficient 2T and
// needs only the first ks(T)*4 multipole coefficients: the triangle
// |a|+|b| <= p), columns = 16 groups.  The row tiles are split over the 4
// waves by a compile-time greedy balance of their k-steps; each wave runs a
// fully unrolled MFMA sequence with its A offsets in registers.
constexpr int m2l_ksteps(int P, int T) { return (nh(P - h_deg(2 * T)) + 3) / 4; }

template <int P>
struct M2LPlan {
  static constexpr int NT = (8 * nh(P) + 15) / 16;
  int n[4] = {0, 0, 0, 0};
  int tile[4][NT] = {};
  int steps[4] = {0, 0, 0, 0};
  int kbmax[4] = {0, 0, 0, 0};
  int base[NT] = {};   // first step of tile T in the natural-order offset table
};

template <int P>
constexpr M2LPlan<P> make_m2l_plan() {
  M2LPlan<P> pl{};
  constexpr int NT = M2LPlan<P>::NT;
  int s = 0;
  for (int T = 0; T < NT; ++T) {
    pl.base[T] = s;
    s += m2l_ksteps(P, T);
  }
  // tiles in natural order have non-increasing k-steps: greedy to the lightest part
  for (int T = 0; T < NT; ++T) {
    int best = 0;
    for (int q = 1; q < 4; ++q)
      if (pl.steps[q] < pl.steps[best]) best = q;
    pl.tile[best][pl.n[best]++] = T;
    pl.steps[best] += m2l_ksteps(P, T);
    if (m2l_ksteps(P, T) > pl.kbmax[best]) pl.kbmax[best] = m2l_ksteps(P, T);
  }
  return pl;
}

// B of one M2L tap in LDS, sB[k][n] (fragment order of the k-steps): thread (n =
// t & 15, v = t >> 4) loads 16-byte vector v of column n's source row and stores each
// value at its coefficient; the waves past the row's last vector have no part in it.
// (With one value per thread and block of the row, as wide as the layout allows up to
// p = 3, all four waves looked up 16 lines per tap: 64^3 at p = 1 FP32 48 us, now
// 33; two ranges of taps.)  A missing or leaf source reads the zero row; the threads of
// vector 0 store a leaf's mass, which was put into LDS with the source table and is
// read with the source (loaded from memory in the tap loop by every thread, it took 40%
// of the kernel at p = 1).
template <typename T, int P>
struct BStage {
  using SL = SymLayout<P, (int)sizeof(T)>;
  typedef typename Vec16<T>::type V;
  static constexpr int VW = TapStage<T, P>::VW, NV = SL::ROW / VW;
  static_assert(SL::NP == 1 && NV % 4 == 0 && NV <= 16, "one vector per thread, whole waves");
  struct Regs {
    V v;
    T m;        // the mass of a leaf
    bool leaf;
  };
  gptr<T> base;
  const int* src;    // [tap][column]
  const T* mass;     // [tap][column]
  int zrow;
  int at[VW];        // sB slots of the thread's values
  __device__ inline void init(const LevelDev& lv, const int* s, const T* m) {
    static constexpr SL sl{};
    const int t = threadIdx.x, n = t & 15, v = t >> 4;
    zrow = lv.nref;
    base = as_global(level_S<T>(lv)) + v * VW;
    src = s;
    mass = m;
    if (v >= NV) return;
#pragma unroll
    for (int i = 0; i < VW; ++i) {
      const int h = sl.coef[v * VW + i];
      at[i] = (h >= 0 ? h : TapStage<T, P>::KP) * 16 + n;
    }
  }
  static __device__ inline constexpr bool part(int wave) { return 4 * wave < NV; }
  // tap k, or none (k < 0); MASS for wave 0, which holds vector 0
  template <bool MASS>
  __device__ inline void load(int k, Regs& r) const {
    const int i = max(k, 0) * 16 + ((int)threadIdx.x & 15), s0 = src[i], sr = k >= 0 ? s0 : -1;
    if (MASS) r.m = mass[i];
    r.v = *(gptr<V>)(base + (size_t)min((uint32_t)sr, (uint32_t)zrow) * SL::ROW);
    if (MASS) r.leaf = threadIdx.x < 16 && sr <= -2;
  }
  template <bool MASS>
  __device__ inline void store(T* sB, const Regs& r) const {
#pragma unroll
    for (int i = 0; i < VW; ++i) sB[at[i]] = MASS && i == 0 && r.leaf ? r.m : r.v[i];
  }
};

// D~ stage copy without a branch around the loads: thread t loads vectors
// t, t + NTH, ... clamped to the last one (stores skip the extra ones).
template <typename T, int P, int NTH>
__device__ inline void load_dstage_nb(int code, const T* __restrict__ Dst, typename Vec16<T>::type* vD) {
  using TS = TapStage<T, P>;
  using V = typename Vec16<T>::type;
  constexpr int NJ = (TS::NDV + NTH - 1) / NTH;
  const int t = threadIdx.x;
  gptr<V> src = (gptr<V>)as_global(Dst + (size_t)(code >> 8) * TS::SDP);
#pragma unroll
  for (int j = 0; j < NJ; ++j) vD[j] = src[min(t + NTH * j, TS::NDV - 1)];
}

// One wave's share of an M2L tile: its row tiles (compile-time plan H) over
// the block's LDS stage of B and of the D~ rows.  The stage of tap k + 2 is
// loaded into registers while the MFMAs of tap k run and stored to LDS after
// those of tap k + 1 (two register sets, two LDS buffers), so a load has two
// taps to land; the sources of every tap of the range were resolved into LDS
// (sSrcT) before the loop.
template <typename T, int P, int H>
__device__ inline void m2l_part(const int32_t* __restrict__ tp, int nt, const int16_t* __restrict__ aoff,
                                const int* sF, T (*sB)[TapStage<T, P>::SB],
                                T (*sD)[TapStage<T, P>::SDP], const BStage<T, P>& bs,
                                const T* __restrict__ Dst, gptr<int32_t> rank0, gmut<T> Lout, int ldl) {
  using TS = TapStage<T, P>;
  using BV = typename BStage<T, P>::Regs;
  using V = typename Vec16<T>::type;
  constexpr int K = TS::K;
  constexpr M2LPlan<P> PL = make_m2l_plan<P>();
  constexpr int NTH = PL.n[H];
  constexpr int NS = PL.steps[H];
  constexpr int KBH = PL.kbmax[H];
  constexpr int ND = (TS::NDV + kBlock - 1) / kBlock;
  const int lane = threadIdx.x & 63, krow = lane >> 4;
  int off[NS > 0 ? NS : 1];
  {
    int s = 0;
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int kb = 0; kb < m2l_ksteps(P, PL.tile[H][i]); ++kb) off[s++] = aoff[(PL.base[PL.tile[H][i]] + kb) * 64 + lane];
  }
  typename Acc4<T>::type acc[NTH > 0 ? NTH : 1], hi = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < NTH; ++i) acc[i] = {0, 0, 0, 0};
  // register sets X (odd taps ahead) and Y; tap 1 goes to X first
  V vDX[ND], vDY[ND];
  BV vBX, vBY;
  // Taps run in pairs; an odd range ends with one empty tap (no source, so B
  // is zero; its D~ stage repeats the last tap's finite rows), so that both
  // steps of a pair and every load run unconditionally.
  const int nt2 = (nt + 1) & ~1;
  {
    const int k1 = nt > 1 ? 1 : 0;
    load_dstage_nb<T, P, kBlock>(tp[k1], Dst, vDX);
    if constexpr (BStage<T, P>::part(H)) bs.template load<H == 0>(nt > 1 ? 1 : -1, vBX);
  }
  // one tap: load tap k + 2 into (vDn, vBn), MFMAs of tap k from LDS buffer
  // b, store tap k + 1 from (vDc, vBc) into buffer b ^ 1
  auto step = [&](int k, int b, V* vDc, const BV& vBc, V* vDn, BV& vBn) {
    const int k2 = k + 2 < nt ? k + 2 : nt - 1;
    load_dstage_nb<T, P, kBlock>(tp[k2], Dst, vDn);
    if constexpr (BStage<T, P>::part(H)) bs.template load<H == 0>(k + 2 < nt ? k2 : -1, vBn);
    __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the MFMAs
    const T* B = sB[b] + lane;
    const T* D = sD[b];
    T bv[KBH > 0 ? KBH : 1];
#pragma unroll
    for (int kb = 0; kb < KBH; ++kb) bv[kb] = B[kb * 64];
    int s = 0;
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int kb = 0; kb < m2l_ksteps(P, PL.tile[H][i]); ++kb) {
        auto& sum = PL.tile[H][i] == 0 && kb > 0 ? hi : acc[i];
        sum = mfma16(D[off[s]], bv[kb], sum);
        ++s;
      }
    if (k + 1 < nt2) {
      store_dstage<T, P, kBlock>(sD[b ^ 1], vDc);
      if constexpr (BStage<T, P>::part(H)) bs.template store<H == 0>(sB[b ^ 1], vBc);
    }
    __syncthreads();
  };
  for (int k = 0; k < nt2; k += 2) {
    step(k, 0, vDX, vBX, vDY, vBY);
    step(k + 1, 1, vDY, vBY, vDX, vBX);
  }
  if (NTH > 0 && PL.tile[H][0] == 0) acc[0] += hi;
  const int F = sF[lane & 15];
  if (F < 0) return;
#pragma unroll
  for (int i = 0; i < NTH; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int R = 16 * PL.tile[H][i] + acc_row<T>(krow, r);
      if ((R >> 3) >= K) continue;
      const int ry = rank0[8 * F + (R & 7)];
      if (ry >= 0) Lout[(size_t)ry * ldl + (R >> 3)] = acc[i][r];
    }
  }
}

// Occupancy floor of k_m2l_taps: told to keep 4 waves per SIMD, the compiler takes 69
// registers at p = 4 FP32 instead of 92 and M2L runs 2 to 4% faster (64^3 + 2% of its
// cells: 133, 137 us); up to p = 3 the times are equal, and the FP64 kernels come out
// the same with any floor that they reach without spilling.
template <typename T>
constexpr int m2l_min_waves() { return sizeof(T) == 4 ? 4 : 1; }

// One block = one tile (16 groups) and one of `nsplit` contiguous tap ranges.
// With nsplit == 1 the sums go to the front of the rows of L; otherwise to the
// level's partial buffer [nsplit][nref][KH], reduced in fixed order by k_l2l,
// which also forms the coefficients that follow from these.
template <typename T, int P>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(m2l_min_waves<T>())))
void k_m2l_taps(const int32_t* __restrict__ tiles, int ntiles, int nsplit,
                                                     const int32_t* __restrict__ taps,
                                                     const int16_t* __restrict__ aoff,
                                                     const LevelDev* __restrict__ lvs, const T* __restrict__ Dst) {
  using TS = TapStage<T, P>;
  using BS = BStage<T, P>;
  constexpr int ND = (TS::NDV + kBlock - 1) / kBlock;
  __shared__ T sB[2][TS::SB];
  __shared__ __align__(16) T sD[2][TS::SDP];
  __shared__ int sF[16];
  __shared__ int sSrcT[kTaps * 16];
  __shared__ T sM[kTaps * 16];
  int* sCB = (int*)sM;  // [16][27], until the sources are known
  __shared__ int sCode[kTaps];
  __shared__ int sNt;
  const int item = xcd_tile(ntiles * nsplit);
  if (item >= ntiles * nsplit) return;
  const int tile = item / nsplit, chunk = item - tile * nsplit;
  int tb, te;
  tap_range(chunk, nsplit, tb, te);
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int32_t* rec = tiles + (size_t)tile * 17;
  const int f = rec[0];
  const LevelDev lv1 = lvs[f - 1];
  const LevelDev lv0 = lvs[f];
  tile_setup(rec, 16, lvs[f - 2], lv1, sF, sCB);
  __syncthreads();
  const int oF = as_global(lv1.refcell)[sF[0]] & 7;
  const int32_t* tpg = taps + oF * kTaps + tb;
  gptr<int32_t> rank1 = as_global(lv1.rank);
  // coefficients past the last one, covered by the last k-step, stay 0
  for (int i = TS::K * 16 + t; i < TS::KP * 16; i += kBlock) sB[0][i] = sB[1][i] = 0;
  // sources of every tap of the range, then the taps with a source (wave 0)
  for (int i = t; i < (te - tb) * 16; i += kBlock) sSrcT[i] = tap_src(tpg[i >> 4], i & 15, sCB, rank1);
  __syncthreads();
  if (w == 0) {
    const int c = compact_taps(te - tb, tpg, sSrcT, sCode);
    if (lane == 0) sNt = c;
  }
  __syncthreads();
  const int nt = sNt;
  const int* tp = sCode;
  for (int i = t; i < nt * 16; i += kBlock) {
    const int sr = sSrcT[i];
    sM[i] = (T)as_global(lv1.mass)[sr <= -2 ? -2 - sr : 0];
  }
  BS bs;
  bs.init(lv1, sSrcT, sM);
  __syncthreads();
  {
    typename Vec16<T>::type vD[ND];
    typename BS::Regs vB;
    load_dstage_nb<T, P, kBlock>(tp[0], Dst, vD);
    if (BS::part(w)) {
      bs.template load<true>(0, vB);
      bs.template store<true>(sB[0], vB);
    }
    store_dstage<T, P, kBlock>(sD[0], vD);
  }
  __syncthreads();
  gmut<T> Lout = as_global_mut(nsplit > 1 ? (T*)lv0.Lpart + (size_t)chunk * lv0.nref * TS::K : level_L<T>(lv0));
  const int ldl = nsplit > 1 ? TS::K : nmi(P);
  gptr<int32_t> rank0 = as_global(lv0.rank);
  // every wave runs the same number of barriers (one per tap)
  switch (w) {
    case 0: m2l_part<T, P, 0>(tp, nt, aoff, sF, sB, sD, bs, Dst, rank0, Lout, ldl); break;
    case 1: m2l_part<T, P, 1>(tp, nt, aoff, sF, sB, sD, bs, Dst, rank0, Lout, ldl); break;
    case 2: m2l_part<T, P, 2>(tp, nt, aoff, sF, sB, sD, bs, Dst, rank0, Lout, ldl); break;
    default: m2l_part<T, P, 3>(tp, nt, aoff, sF, sB, sD, bs, Dst, rank0, Lout, ldl); break;
  }
}

// ---------------------------------------------------------------------------
// M2L sums from p = 5 (Alg. 3 without the ShiftLocal term, which the L2L chain adds
// afterwards), by the reflections of the axes as in M2P: with
//   U_chi[a] = sum over an orbit's sources of chi(sigma) sigma^a S_sigma[a]
// the children's local expansions are
//   L_o[b] = tau^b sum_chi chi(tau) Lambda_chi[b],
//   Lambda_chi[b] = sum over orbits and |a| + |b| <= p of E_(chi ^ par b)[a + b] U_chi[a],
// par b the parities of b.  56 orbits x 8 characters x 532 products per group at
// p = 6 instead of 189 sources x 8 children x 532.
//
// A block takes NC groups of one parity class and a range of the orbits; wave chi
// forms Lambda_chi of all its columns.  Per orbit, thread (pass, block q, column)
// holds block q (SymLayout) of the orbit's sources of one column; all coefficients
// of a block have one parity, so butterflies in registers make the distinct U of
// the orbit (one per character of its reflected axes), which go to LDS in the
// order of the products' k-steps.  The loads of the next orbit are in flight
// during the products of one.  The E rows of an orbit (8 x K values, with the
// signs of the class) are staged in LDS; a lane gathers its A operand from there
// through offsets that depend on the character only (registers).
// Products, FP32: 4 x 4 x 1 blocks (16 per instruction: 4 k x 4 column quads), the
// row quad picked by the broadcast of A, so that a row quad of degree n runs only
// the k-steps below degree p - n: 46 x 256 products per character and column tile
// at p = 6 where 16-row tiles take 18 x 1024.  FP64: 16 x 16 x 4.
// In FP32 the first k-step (monopole and dipole terms, by far the largest) sums
// into an accumulator of its own in the lowest rows: the terms of orders >= 2 are
// many, and below half a unit in the last place of the running sum they were
// rounded away on one side (mean error of the potential 7e-7 at p = 6, 0.4e-7 apart).
// Bound by instruction issue: one block of 8 waves per CU, whose butterflies,
// addresses and LDS traffic cost about as much as the products, and the barrier of
// every orbit.  A wider tile (or a second block) does not fit the registers (253 at
// p = 6 FP32); a second orbit's loads in flight changed nothing.  Tap by tap on all
// coefficients / on the folded ones / by orbits: 8.08M leaves p = 6 FP32 3.9 / 2.60 /
// 2.04 ms; the last two, 287,680 leaves p = 6 FP64 272 / 184 us, 8 hierarchies p = 8
// FP32 720 / 457 us.
__device__ inline f32x4 mfma4q(int quad, float a, float b, f32x4 c) {
  switch (quad) {  // constant at every call
    case 0: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 2, 0, 0);
    case 1: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 2, 1, 0);
    case 2: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 2, 2, 0);
    default: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 2, 3, 0);
  }
}

template <typename T, int P, int NC>
struct M2L {
  using SL = SymLayout<P, (int)sizeof(T)>;
  using V16 = typename Vec16<T>::type;
  static constexpr int CP = SL::CP, NP = SL::NP, ROW = SL::ROW;
  static constexpr int KH = nh(P), KB = (KH + 3) / 4, RT = (KH + 15) / 16;
  static constexpr int CT = NC / 16;
  static constexpr bool QUADS = sizeof(T) == 4;
  static constexpr int UT = KB * 64 + 16;             // U of one column tile (the tiles 16 banks apart)
  static constexpr int UP = CT * UT + 64;             // U of one character, then places for the unused slots
  static constexpr int ES = sym_es(P), EL = sym_elen(P, (int)sizeof(T));
  static constexpr int NIT = NP * 16 * NC;            // (pass, block, column)
  static constexpr int NI = (NIT + kM2LBlock - 1) / kM2LBlock;
  static constexpr int VW = 16 / (int)sizeof(T), NEV = EL / VW;  // vectors of the E rows
  static constexpr int NE = (NEV + kM2LBlock - 1) / kM2LBlock;
  static constexpr int SRC = 216 * NC;
  // two sets of U and E where they fit the LDS
  static constexpr int NBUF = 2 * (8 * UP + EL) * (int)sizeof(T) + (SRC + 9 * NC) * 4 <= 160 * 1024 ? 2 : 1;
  static_assert(NIT % 64 == 0 && kM2LBlock % (16 * NC) == 0, "whole waves, one block q per thread");
  typedef typename VecN<T, CP>::type V;
  struct Lds {  // E first: the gathers' places and the buffer's fit the instruction's offset
    T e[NBUF][EL];
    int src[SRC];       // [m][neighbour][column]: rank, or -2 - cell of a leaf, or -1
    int F[NC];
    int rank0[8 * NC];  // [column][child]
    T u[NBUF][8 * UP];
  };
  static constexpr int LS = NC + 1;  // Lambda's row stride in LDS
  static_assert(8 * KH * LS <= NBUF * 8 * UP, "Lambda in the place of U");
  // k-steps of the row quad i of row tile r (0: no rows)
  static constexpr int ks(int r, int i) { return 16 * r + 4 * i < KH ? (nh(P - h_deg(16 * r + 4 * i)) + 3) / 4 : 0; }
  static constexpr int steps() {
    int s = 0;
    for (int r = 0; r < RT; ++r) s += ks(r, 0);
    return s;
  }
  static constexpr int NS = steps();

  Lds& l;
  gptr<T> S;
  gptr<double> mass1;
  const T* __restrict__ symE;
  sptr<uint64_t> taps;
  sptr<int> var;
  uint64_t code;         // neighbours of the next orbit's sources, a byte each
  int vr;                // and its variant
  int zrow, col, q, s0, wave;
  bool on;               // the thread has a first item
  T sg[3];
  int at[NI * CP];       // places in U of the thread's values
  struct Regs {          // an orbit on its way
    V v[NI][8];
    double mm[8];
    unsigned leaf;
    V16 e[NE];
  };

  static __device__ inline int set_of(int g) {
    const int m = g / 7;
    return sym_axes(sym_set(m, g - 7 * m));
  }
  // sources 2^(NB-1) .. 2^NB - 1 of an orbit (NB = 0: source 0).  The steps of nb
  // reflections nest, so that a value has one register whatever the orbit: copies
  // behind a branch would wait for the loads
  template <int NB>
  __device__ inline void load_rows(int nb, const int* sc, Regs& r) const {
    if (nb < NB) return;
    constexpr int I0 = NB ? 1 << (NB - 1) : 0, I1 = 1 << NB;
#pragma unroll
    for (int i = I0; i < I1; ++i) {
      gptr<T> row = S + (size_t)min((uint32_t)sc[i], (uint32_t)zrow) * ROW;  // no source or a leaf: the zero row
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const int s = k * (kM2LBlock / (16 * NC));
        r.v[k][i] = load_vec<T, CP>(row + (k == 0 || s0 + s < NP ? s : 0) * kSymBlocks * CP);
      }
    }
    if (wave == 0) {  // its lanes hold the monopoles
#pragma unroll
      for (int i = I0; i < I1; ++i) {
        r.mm[i] = mass1[sc[i] <= -2 ? -2 - sc[i] : 0];
        r.leaf |= (unsigned)(sc[i] <= -2) << i;
      }
    }
    if constexpr (NB < 3) load_rows<NB + 1>(nb, sc, r);
  }
  // scalars of orbit g, read one orbit ahead of their use
  __device__ inline void next(int g) {
    code = taps[g];
    vr = var[g];
  }
  // loads of orbit g
  __device__ inline void load(int g, Regs& r) const {
    gptr<V16> e = (gptr<V16>)as_global(symE + (size_t)vr * EL);
#pragma unroll
    for (int k = 0; k < NE; ++k) r.e[k] = e[min((int)threadIdx.x + kM2LBlock * k, NEV - 1)];
    if (on) {
      r.leaf = 0;
      const int base = g / 7 * 27 * NC + col;
      int sc[8];  // all at once (bytes past the orbit's sources are 0)
#pragma unroll
      for (int i = 0; i < 8; ++i) sc[i] = l.src[base + ((int)(code >> (8 * i)) & 31) * NC];
      load_rows<0>(sym_bits(set_of(g)), sc, r);
    }
  }
  template <int B>
  static __device__ inline void stage(Regs& r, int i0, int n, T s) {  // butterflies of index bit B on values i0 .. i0 + n - 1
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
      for (int i = i0; i < i0 + n; ++i)
        if (!(i >> B & 1)) {
          const V x = r.v[k][i], y = r.v[k][i | 1 << B];
#pragma unroll
          for (int e = 0; e < CP; ++e) {
            r.v[k][i][e] = x[e] + s * y[e];
            r.v[k][i | 1 << B][e] = x[e] - s * y[e];
          }
        }
  }
  __device__ inline T axis_sign(int rest) const {  // of the lowest axis of the set
    const T x0 = sg[0], x1 = sg[1], x2 = sg[2];
    return rest & 1 ? x0 : rest & 2 ? x1 : x2;
  }
  template <int I0, int I1>
  __device__ inline void put_u(T* u, const Regs& r) const {
#pragma unroll
    for (int k = 0; k < NI; ++k)
      if (k == 0 || s0 + k * (kM2LBlock / (16 * NC)) < NP) {
#pragma unroll
        for (int i = I0; i < I1; ++i)
#pragma unroll
          for (int e = 0; e < CP; ++e) u[i * UP + at[k * CP + e]] = r.v[k][i][e];
      }
  }
  // the loaded orbit g into LDS
  __device__ inline void put(int g, int buf, Regs& r) const {
#pragma unroll
    for (int k = 0; k < NE; ++k)
      if ((int)threadIdx.x + kM2LBlock * k < NEV) ((V16*)l.e[buf])[threadIdx.x + kM2LBlock * k] = r.e[k];
    if (!on) return;
    T* u = l.u[buf];
    const int pt = set_of(g), nb = sym_bits(pt);
    if (wave == 0) {
      const unsigned lf = (int)threadIdx.x < NC ? r.leaf : 0;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (lf >> i & 1) r.v[0][i][0] = (T)r.mm[i];
    }
    const T t0 = axis_sign(pt), t1 = axis_sign(pt & (pt - 1)), t2 = sg[2];
    if (nb >= 1) {
      stage<0>(r, 0, 2, t0);
      if (nb >= 2) {
        stage<0>(r, 2, 2, t0);
        stage<1>(r, 0, 4, t1);
        if (nb >= 3) {
          stage<0>(r, 4, 4, t0);
          stage<1>(r, 4, 4, t1);
          stage<2>(r, 0, 8, t2);
          put_u<4, 8>(u, r);
        }
        put_u<2, 4>(u, r);
      }
      put_u<1, 2>(u, r);
    }
    put_u<0, 1>(u, r);
  }
};

// One block = one tile and one of `nsplit` contiguous ranges of the orbits.  With
// nsplit == 1 the sums go to the front of the rows of L; otherwise to the level's
// partial buffer [nsplit][nref][KH], reduced in fixed order by k_l2l, which also
// forms the coefficients that follow from these.
template <typename T, int P, int NC>
__global__ __launch_bounds__(kM2LBlock)
void k_m2l(const int32_t* __restrict__ tiles, int ntiles, int nsplit, const int8_t* __restrict__ taps,
           const int* __restrict__ var, const int16_t* __restrict__ aoff, const LevelDev* __restrict__ lvs,
           const T* __restrict__ symE) {
  using ML = M2L<T, P, NC>;
  using SL = typename ML::SL;
  static constexpr SL sl{};
  constexpr int CT = ML::CT, RT = ML::RT, KB = ML::KB, KH = ML::KH;
  __shared__ __align__(16) typename ML::Lds lds;
  const int item = xcd_tile(ntiles * nsplit);
  if (item >= ntiles * nsplit) return;
  const int tile = item / nsplit, chunk = item - tile * nsplit;
  const int t = threadIdx.x, lane = t & 63, chi = __builtin_amdgcn_readfirstlane(t >> 6);
  const int32_t* rec = tiles + (size_t)tile * (NC + 1);
  const int f = rec[0];
  const LevelDev lv0 = lvs[f], lv1 = lvs[f - 1], lv2 = lvs[f - 2];
  if (t < NC) lds.F[t] = rec[1 + t];
  for (int i = t; i < ML::NBUF * 8 * ML::UP; i += kM2LBlock) (&lds.u[0][0])[i] = 0;  // k-steps past the last coefficient
  __syncthreads();
  gptr<int32_t> refcell1 = as_global(lv1.refcell);
  const int C = __builtin_amdgcn_readfirstlane(refcell1[lds.F[0]] & 7);
  // sources of the columns: the 8 children of each neighbour of their fathers
  for (int i = t; i < 27 * NC; i += kM2LBlock) {
    const int e = i / NC, F = lds.F[i - e * NC];
    const int Q = F >= 0 ? as_global(lv2.nbr)[(size_t)(refcell1[F] >> 3) * 27 + e] : -1;
    const int rQ = Q >= 0 ? as_global(lv2.rank)[Q] : -1;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    gptr<i32x4> rk = (gptr<i32x4>)(as_global(lv1.rank) + 8 * max(rQ, 0));
    const i32x4 lo = rk[0], up = rk[1];
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      const int r = o < 4 ? lo[o & 3] : up[o & 3];
      lds.src[(o ^ C) * 27 * NC + i] = rQ < 0 ? -1 : r >= 0 ? r : -2 - (8 * rQ + o);
    }
  }
  for (int i = t; i < 8 * NC; i += kM2LBlock) {
    const int F = lds.F[i >> 3];
    lds.rank0[i] = F >= 0 ? as_global(lv0.rank)[8 * F + (i & 7)] : -1;
  }
  ML m{lds};
  m.S = as_global(level_S<T>(lv1)) + (t / (16 * NC) * kSymBlocks + (t / NC & 15)) * ML::CP;
  m.mass1 = as_global(lv1.mass);
  m.symE = symE;
  m.wave = chi;
  m.taps = (sptr<uint64_t>)taps + C * kSymOrbits;
  m.var = (sptr<int>)var + C * kSymOrbits;
  m.zrow = lv1.nref;
  m.col = t % NC;
  m.q = t / NC & 15;
  m.s0 = t / (16 * NC);
  m.on = 64 * chi < ML::NIT;
  {
    const int par = sl.par[m.q];
#pragma unroll
    for (int i = 0; i < 3; ++i) m.sg[i] = par >> i & 1 ? (T)-1 : (T)1;
#pragma unroll
    for (int k = 0; k < ML::NI; ++k) {
      const int s = m.s0 + k * (kM2LBlock / (16 * NC));
#pragma unroll
      for (int e = 0; e < ML::CP; ++e) {
        const int h = s < ML::NP ? sl.coef[(s * kSymBlocks + m.q) * ML::CP + e] : -1;
        m.at[k * ML::CP + e] = h < 0 ? CT * ML::UT + lane : (m.col >> 4) * ML::UT + (h >> 2) * 64 + (h & 3) * 16 + (m.col & 15);
      }
    }
  }
  int off[ML::NS];
#pragma unroll
  for (int i = 0; i < ML::NS; ++i) off[i] = as_global(aoff)[(chi * ML::NS + i) * 64 + lane];
  typename Acc4<T>::type acc[RT][ML::QUADS ? 4 : 1][CT], hi[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    hi[c] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < (ML::QUADS ? 4 : 1); ++i) acc[r][i][c] = {0, 0, 0, 0};
  }
  const int g0 = chunk * kSymOrbits / nsplit, g1 = (chunk + 1) * kSymOrbits / nsplit;
  m.next(g0);
  typename ML::Regs rg;
  rg.leaf = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    rg.mm[i] = 0;
#pragma unroll
    for (int k = 0; k < ML::NI; ++k) rg.v[k][i] = typename ML::V{};
  }
  __syncthreads();
  m.load(g0, rg);
  m.next(min(g0 + 1, g1 - 1));
  m.put(g0, 0, rg);
  __syncthreads();
  auto step = [&](int g, int buf) {
    if (g + 1 < g1) m.load(g + 1, rg);
    m.next(min(g + 2, g1 - 1));
    __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the products
    // the character restricted to the orbit's axes
    const int pt = ML::set_of(g);
    int u = 0, bit = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (pt >> i & 1) u |= (chi >> i & 1) << bit++;
    const T* U = lds.u[buf] + u * ML::UP + lane;
    const T* E = lds.e[buf];
    int s = 0;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (ML::NI > 1 && kb % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // LDS reads hoisted further spill
      T b[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) b[c] = U[c * ML::UT + kb * 64];
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        if (kb >= ML::ks(r, 0)) continue;
        const T a = E[off[s++]];
        if constexpr (ML::QUADS) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (kb < ML::ks(r, i)) {
#pragma unroll
              for (int c = 0; c < CT; ++c) {
                auto& sum = r == 0 && i == 0 && kb > 0 ? hi[c] : acc[r][i][c];
                sum = mfma4q(i, a, b[c], sum);
              }
            }
        } else {
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[r][0][c] = mfma16(a, b[c], acc[r][0][c]);
        }
      }
    }
    if (ML::NBUF == 1) __syncthreads();
    if (g + 1 < g1) m.put(g + 1, ML::NBUF == 2 ? buf ^ 1 : 0, rg);
    __syncthreads();
  };
  for (int g = g0; g < g1; ++g) {
    step(g, 0);
    if (ML::NBUF == 2 && ++g < g1) step(g, 1);
  }
  // Lambda to LDS, [chi][b][column]
  T* lam = &lds.u[0][0] + chi * KH * ML::LS;
  const int kq = lane >> 4;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    if constexpr (ML::QUADS) {
      acc[0][0][c] += hi[c];
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (ML::ks(r, i) == 0) continue;
          // sum over the four k of the blocks: lane group kq keeps row kq
          const auto x = acc[r][i][c];
          const bool up = kq & 2, odd = kq & 1;
          T y0 = up ? x[2] : x[0], y1 = up ? x[3] : x[1];
          y0 += __shfl_xor(up ? x[0] : x[2], 32, 64);
          y1 += __shfl_xor(up ? x[1] : x[3], 32, 64);
          const T z = (odd ? y1 : y0) + __shfl_xor(odd ? y0 : y1, 16, 64);
          const int h = 16 * r + 4 * i + kq;
          if (h < KH) lam[h * ML::LS + 16 * c + (lane & 15)] = z;
        }
    } else {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int h = 16 * r + acc_row<T>(kq, j);
          if (h < KH) lam[h * ML::LS + 16 * c + (lane & 15)] = acc[r][0][c][j];
        }
    }
  }
  __syncthreads();
  gmut<T> Lout = as_global_mut(nsplit > 1 ? (T*)lv0.Lpart + (size_t)chunk * lv0.nref * KH : level_L<T>(lv0));
  const int ldl = nsplit > 1 ? KH : nmi(P);
  for (int i = t; i < KH * NC; i += kM2LBlock) {
    const int n = i / KH, h = i - n * KH;
    T x[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) x[c] = (&lds.u[0][0])[(c * KH + h) * ML::LS + n];
    // characters -> children (index y = ~o)
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (!(c & bit)) {
          const T y = x[c], z = x[c | bit];
          x[c] = y + z;
          x[c | bit] = y - z;
        }
    const int par = h_parity(h);
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      const int ry = lds.rank0[8 * n + (7 - y)];
      if (ry >= 0) Lout[(size_t)ry * ldl + h] = __popc(par & y) & 1 ? -x[y] : x[y];
    }
  }
}

// ---------------------------------------------------------------------------
// Leaf evaluation at level l (Alg. 4): far field (L2P of L[F]) and near field
// (P2P from the level-l leaves among the children of F's 27 neighbours and
// from the neighbours that are leaves one level coarser).  For every group
// these are one fixed linear map of the same gathered inputs (the candidates'
// masses, L[F]), so 16 groups are one product [32 x near_cols] . [near_cols x
// 16] on 16x16x4 MFMA: rows c * 8 + o (phi, ax, ay, az of child o), columns
// in the order of the operator table nearA.  Lane (n = lane & 15, g = lane >>
// 4) gathers column n's inputs for steps 4 kb + g straight into registers.
// The intermediate-field partials (k_m2p) and the partial of the refined near
// cells (near M2P and nearest-field P2P, k_near_m2p; zero for groups without
// such cells) are added in FP64 and the sums scaled to physical units.  One
// block per 16 groups of the level's group list; its 4 waves take a quarter
// of the operator columns each (more loads in flight per tile), and wave 0
// adds the other waves' accumulators in order.
template <typename T, int P, int W>
__device__ inline void near_part(int lane, int F, const int* __restrict__ sCB, gptr<double> mass0,
                                 gptr<double> mass1, const T* __restrict__ Lpar, const T* __restrict__ nearA,
                                 typename Acc4<T>::type& acc0, typename Acc4<T>::type& acc1) {
  using V = typename Vec16<T>::type;
  constexpr int K = nmi(P);
  constexpr int VW = 16 / (int)sizeof(T);
  constexpr int NQ = near_ksteps(P) / VW;
  constexpr int Q0 = W * NQ / 4, Q1 = (W + 1) * NQ / 4;
  constexpr int C0 = kNearLeafCols, C1 = kNearLeafCols + kNearCoarseCols;
  const int n = lane & 15, g = lane >> 4;
  // B: column n's inputs for steps 4 kb + g (refined cells hold mass 0; every
  // load has a valid address, the value is selected afterwards)
  T bv[(Q1 - Q0) * VW + 1];
#pragma unroll
  for (int i = 0; i < (Q1 - Q0) * VW; ++i) {
    const int k = 4 * (Q0 * VW + i) + g;
    T v = 0;
    if (k < C0) {
      const int cb = sCB[n * 27 + (k >> 3)];
      const double m = mass0[cb >= 0 ? cb + (k & 7) : 0];
      v = cb >= 0 ? (T)m : (T)0;
    } else if (k < C1) {
      const int cb = sCB[n * 27 + (k - C0)];
      const double m = mass1[cb <= -2 ? -2 - cb : 0];
      v = cb <= -2 ? (T)m : (T)0;
    } else if (k < C1 + K) {
      if (Lpar) {
        const T l = as_global(Lpar)[(size_t)(F >= 0 ? F : 0) * K + (k - C1)];
        v = F >= 0 ? l : (T)0;
      }
    }
    bv[i] = v;
  }
  gptr<V> A = (gptr<V>)as_global(nearA);
#pragma unroll
  for (int q = Q0; q < Q1; ++q) {
    const V a0 = A[(size_t)q * 64 + lane];
    const V a1 = A[(size_t)(NQ + q) * 64 + lane];
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      acc0 = mfma16(a0[j], bv[(q - Q0) * VW + j], acc0);
      acc1 = mfma16(a1[j], bv[(q - Q0) * VW + j], acc1);
    }
  }
}

template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_near(const int32_t* __restrict__ grp, int ngrp, LevelDev lv1, LevelDev lv0,
                                                 const T* __restrict__ nearA, const T* __restrict__ Lpar,
                                                 const T* __restrict__ part, const T* __restrict__ nmp, double G,
                                                 double h, double cself, double* __restrict__ phi,
                                                 double* __restrict__ acc) {
  static_assert(kBlock == 256, "four waves split the operator columns");
  static_assert(near_ksteps(P) % (16 / (int)sizeof(T)) == 0, "near operator vectors");
  __shared__ int sF[16];
  __shared__ int sCB[16 * 27];
  __shared__ T sAcc[3][8][64];
  const int ntiles = (ngrp + 15) / 16;
  const int tile = xcd_tile(ntiles);
  if (tile >= ntiles) return;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  if (t < 16) sF[t] = 16 * tile + t < ngrp ? grp[16 * tile + t] : -1;
  __syncthreads();
  // per group and neighbour e: child base 8 rq (refined neighbour), -2 - q
  // (leaf neighbour q), or -1 (outside the box)
  gptr<int32_t> nbr1 = as_global(lv1.nbr), rank1 = as_global(lv1.rank);
  for (int i = t; i < 16 * 27; i += kBlock) {
    const int c = i / 27, e = i - 27 * c;
    const int F = sF[c];
    int v = -1;
    if (F >= 0) {
      const int q = nbr1[(size_t)F * 27 + e];
      if (q >= 0) {
        const int rq = rank1[q];
        v = rq >= 0 ? 8 * rq : -2 - q;
      }
    }
    sCB[i] = v;
  }
  __syncthreads();
  const int n = lane & 15, g = lane >> 4;
  const int F = sF[n];
  gptr<double> mass0 = as_global(lv0.mass), mass1 = as_global(lv1.mass);
  typename Acc4<T>::type acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  switch (w) {
    case 0: near_part<T, P, 0>(lane, F, sCB, mass0, mass1, Lpar, nearA, acc0, acc1); break;
    case 1: near_part<T, P, 1>(lane, F, sCB, mass0, mass1, Lpar, nearA, acc0, acc1); break;
    case 2: near_part<T, P, 2>(lane, F, sCB, mass0, mass1, Lpar, nearA, acc0, acc1); break;
    default: near_part<T, P, 3>(lane, F, sCB, mass0, mass1, Lpar, nearA, acc0, acc1); break;
  }
  if (w > 0)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sAcc[w - 1][r][lane] = acc0[r];
      sAcc[w - 1][4 + r][lane] = acc1[r];
    }
  __syncthreads();
  if (w > 0 || F < 0) return;
#pragma unroll
  for (int v = 0; v < 3; ++v)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc0[r] += sAcc[v][r][lane];
      acc1[r] += sAcc[v][4 + r][lane];
    }
  gptr<int32_t> rank0 = as_global(lv0.rank), slot0 = as_global(lv0.slot);
  const double sp = G / h, sa = G / (h * h);
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int R = 16 * tt + acc_row<T>(g, r);
      const int c = R >> 3, cell = 8 * F + (R & 7);
      if (rank0[cell] >= 0) continue;  // refined child: not a target
      double v = (double)(tt ? acc1[r] : acc0[r]);
      if (part)
        for (int s = 0; s < lv1.npart; ++s) v += (double)as_global(part)[((size_t)s * lv1.nref + F) * 32 + R];
      if (nmp) v += (double)as_global(nmp)[(size_t)F * 32 + R];
      const int sl = slot0[cell];
      if (c == 0)
        phi[sl] = sp * (v - cself * mass0[cell]);  // optional self term of the leaf's own mass
      else
        acc[3 * (size_t)sl + c - 1] = sa * v;
    }
}

// Refined level-l cells among the near candidates of a group (children of
// F's 27 neighbours): M2P from those that do not touch the target (Alg. 4) and
// P2P from the 8 children of those that do (nearest field, Sec. 3.2; the
// children are leaves by the grading rule).  One block per group: the refined
// candidates are compacted into LDS (ballot per wave, in candidate order),
// thread (o = t & 7, j = t >> 3) takes target o and every 32nd candidate from
// j, first for the M2P and then, in a separate loop, for the nearest field
// (so that threads on one path do not wait for the other); partial sums are
// reduced by shuffles within a wave and in order across the waves, and
// threads 0..7 write nmp[F][c * 8 + o] (target-level units), read by k_near.
// Every child o is evaluated (refined ones are not read).
template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_near_m2p(const int32_t* __restrict__ grp, int ngrp, LevelDev lv1,
                                                     LevelDev lv0, LevelDev lvp, const T* __restrict__ Dsame,
                                                     const T* __restrict__ S0, T* __restrict__ nmp) {
  static_assert(kBlock == 256, "one candidate per thread in the compaction");
  constexpr int K = nmi(P);
  constexpr int NW = kBlock / 64;
  constexpr int NJ = kBlock / 8;
  __shared__ int s_c[216];
  __shared__ int s_rn[216];
  __shared__ int s_cnt[NW];
  __shared__ T s_red[NW][4][8];
  const int gi = blockIdx.x;
  if (gi >= ngrp) return;
  const int F = grp[gi];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  int rn = -1;
  if (t < 216) {
    const int q = lv1.nbr[(size_t)F * 27 + (t >> 3)];
    if (q >= 0) {
      const int rq = lv1.rank[q];
      if (rq >= 0) rn = lv0.rank[8 * rq + (t & 7)];
    }
  }
  const uint64_t m = __ballot(rn >= 0);
  if (lane == 0) s_cnt[w] = __popcll(m);
  __syncthreads();
  int base = 0, nlist = 0;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    base += v < w ? s_cnt[v] : 0;
    nlist += s_cnt[v];
  }
  if (rn >= 0) {
    const int pos = base + __popcll(m & ((1ull << lane) - 1ull));
    s_c[pos] = t;
    s_rn[pos] = rn;
  }
  __syncthreads();
  const int o = t & 7, j = t >> 3;
  T sum[4] = {0, 0, 0, 0};
  for (int i = j; i < nlist; i += NJ) {
    const int c = s_c[i], e = c >> 3, op = c & 7;
    const int tx = o_axis(o, 0) - 2 * e_axis(e, 0) - o_axis(op, 0);
    const int ty = o_axis(o, 1) - 2 * e_axis(e, 1) - o_axis(op, 1);
    const int tz = o_axis(o, 2) - 2 * e_axis(e, 2) - o_axis(op, 2);
    if (max(abs(tx), max(abs(ty), abs(tz))) <= 1) continue;
    m2p_row<T, P>(Dsame + (size_t)d_index(tx, ty, tz) * K, S0 + (size_t)s_rn[i] * src_row(P, (int)sizeof(T)), sum);
  }
  gptr<double> massp = as_global(lvp.mass);
  for (int i = j; i < nlist; i += NJ) {
    const int c = s_c[i], e = c >> 3, op = c & 7;
    const int tx = o_axis(o, 0) - 2 * e_axis(e, 0) - o_axis(op, 0);
    const int ty = o_axis(o, 1) - 2 * e_axis(e, 1) - o_axis(op, 1);
    const int tz = o_axis(o, 2) - 2 * e_axis(e, 2) - o_axis(op, 2);
    if (max(abs(tx), max(abs(ty), abs(tz))) > 1) continue;
    double mc[8];
#pragma unroll
    for (int o2 = 0; o2 < 8; ++o2) mc[o2] = massp[8 * s_rn[i] + o2];
#pragma unroll
    for (int o2 = 0; o2 < 8; ++o2)
      p2p<T>((T)tx - ((T)o_axis(o2, 0) - (T)0.5) * (T)0.5, (T)ty - ((T)o_axis(o2, 1) - (T)0.5) * (T)0.5,
             (T)tz - ((T)o_axis(o2, 2) - (T)0.5) * (T)0.5, (T)mc[o2], sum);
  }
#pragma unroll
  for (int d = 8; d <= 32; d <<= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) sum[c] += __shfl_xor(sum[c], d, 64);
  if (lane < 8)
#pragma unroll
    for (int c = 0; c < 4; ++c) s_red[w][c][o] = sum[c];
  __syncthreads();
  if (t < 8)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      T v = 0;
#pragma unroll
      for (int u = 0; u < NW; ++u) v += s_red[u][c][o];
      nmp[(size_t)F * 32 + c * 8 + o] = v;
    }
}

// Stale trees advanced to the solve's time: each slot's level is found by a
// scan of the (at most 21) level offsets.
__global__ void k_drift(DriftLevels d, const double* __restrict__ m, const double* __restrict__ rate,
                        double* __restrict__ out, int64_t nslots) {
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < nslots; s += (int64_t)gridDim.x * blockDim.x) {
    int i = 0;
    while (i + 1 < d.n && s >= d.off[i + 1]) ++i;
    const double dt = d.dt[i];
    out[s] = dt != 0.0 ? m[s] + dt * rate[s] : m[s];
  }
}

// ---------------------------------------------------------------------------
// launchers

hipError_t launch_drift(const DriftLevels& d, const double* m, const double* rate, double* out, int64_t nslots,
                        hipStream_t st) {
  if (nslots <= 0) return hipSuccess;
  const int blocks = (int)std::min<int64_t>((nslots + 255) / 256, 8192);
  hipLaunchKernelGGL(k_drift, dim3(blocks), dim3(256), 0, st, d, m, rate, out, nslots);
  return hipGetLastError();
}

template <typename T>
static hipError_t m2p_dispatch(int p, const MfmaTiles& mt, int t0, int n, int nsplit, const MfmaTables& tabs,
                               const LevelDev* lvs, const T* symA, hipStream_t st) {
  const int items = n * nsplit;
  const dim3 grid(8 * ((items + 7) / 8)), block(kBlock);
  if (mt.nc != m2p_cols(p, (int)sizeof(T)) || nsplit < 1 || nsplit > kSymOrbits) return hipErrorInvalidValue;
  const int32_t* tl = mt.tiles + (size_t)t0 * (mt.nc + 1);
  switch (p) {
#define AFMM_M2P(PP)                                                                                \
  case PP:                                                                                          \
    hipLaunchKernelGGL((k_m2p<T, PP>), grid, block, 0, st, tl, n, nsplit, tabs.symtaps, lvs, symA); \
    break;
    AFMM_M2P(1) AFMM_M2P(2) AFMM_M2P(3) AFMM_M2P(4) AFMM_M2P(5) AFMM_M2P(6) AFMM_M2P(7) AFMM_M2P(8)
#undef AFMM_M2P
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_m2p(int p, bool fp32, const MfmaTiles& mt, int t0, int n, int nsplit, const MfmaTables& tabs,
                      const LevelDev* lvs, const TablesDev<float>& t32, const TablesDev<double>& t64,
                      hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (fp32) return m2p_dispatch<float>(p, mt, t0, n, nsplit, tabs, lvs, t32.symA, st);
  return m2p_dispatch<double>(p, mt, t0, n, nsplit, tabs, lvs, t64.symA, st);
}

template <typename T>
static hipError_t m2l_dispatch(int p, const MfmaTiles& mt, int t0, int n, int nsplit, const MfmaTables& tabs,
                               const LevelDev* lvs, const TablesDev<T>& td, hipStream_t st) {
  const int items = n * nsplit;
  const dim3 grid(8 * ((items + 7) / 8));
  // tiles of this order and precision, or the narrow ones of a level solve's short chain
  const bool narrow = mt.nc == 16 && m2l_cols(p, (int)sizeof(T)) != 16;
  if ((mt.nc != m2l_cols(p, (int)sizeof(T)) && !narrow) || nsplit < 1 || nsplit > 21) return hipErrorInvalidValue;
  const int32_t* tl = mt.tiles + (size_t)t0 * (mt.nc + 1);
  switch (p) {
#define AFMM_M2L(PP)                                                                                              \
  case PP:                                                                                                        \
    if constexpr (m2l_by_taps(PP)) {                                                                              \
      hipLaunchKernelGGL((k_m2l_taps<T, PP>), grid, dim3(kBlock), 0, st, tl, n, nsplit, tabs.taps, tabs.m2l_off,  \
                         lvs, td.Dstage);                                                                         \
    } else if (narrow) {                                                                                          \
      hipLaunchKernelGGL((k_m2l<T, PP, 16>), grid, dim3(kM2LBlock), 0, st, tl, n, nsplit, tabs.symtaps,           \
                         tabs.symvar, tabs.m2l_off, lvs, td.symE);                                                \
    } else {                                                                                                      \
      hipLaunchKernelGGL((k_m2l<T, PP, m2l_cols(PP, (int)sizeof(T))>), grid, dim3(kM2LBlock), 0, st, tl, n,       \
                         nsplit, tabs.symtaps, tabs.symvar, tabs.m2l_off, lvs, td.symE);                          \
    }                                                                                                             \
    break;
    AFMM_M2L(1) AFMM_M2L(2) AFMM_M2L(3) AFMM_M2L(4) AFMM_M2L(5) AFMM_M2L(6) AFMM_M2L(7) AFMM_M2L(8)
#undef AFMM_M2L
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_m2l(int p, bool fp32, const MfmaTiles& mt, int t0, int n, int nsplit, const MfmaTables& tabs,
                      const LevelDev* lvs, const TablesDev<float>& t32, const TablesDev<double>& t64, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (fp32) return m2l_dispatch<float>(p, mt, t0, n, nsplit, tabs, lvs, t32, st);
  return m2l_dispatch<double>(p, mt, t0, n, nsplit, tabs, lvs, t64, st);
}

template <typename T, typename TL>
static hipError_t l2l_dispatch(int p, const int32_t* grp, int ngrp, const TL* Lpar, const int32_t* rank0, T* Lout,
                               const T* Lpart, int nsplit, size_t stride, const T* w, const CommonDev& cm,
                               hipStream_t st) {
  const dim3 grid(ngrp), block(kBlock);
  if (nsplit < 1 || nsplit > 24) return hipErrorInvalidValue;
  const int ns = nsplit == 1 ? 0 : nsplit <= 8 ? 1 : 2;  // split bucket: 1, 8 or 24 partials
  switch (p * 3 + ns) {
#define AFMM_L2L(PP, NB, NSV)                                                                                    \
  case PP * 3 + NB:                                                                                              \
    hipLaunchKernelGGL((k_l2l<T, TL, PP, NSV>), grid, block, 0, st, grp, Lpar, rank0, Lout, Lpart, nsplit,       \
                       stride, w, cm.sumidx, cm.mi);                                                             \
    break;
#define AFMM_L2L3(PP) AFMM_L2L(PP, 0, 1) AFMM_L2L(PP, 1, 8) AFMM_L2L(PP, 2, 24)
    AFMM_L2L3(1) AFMM_L2L3(2) AFMM_L2L3(3) AFMM_L2L3(4) AFMM_L2L3(5) AFMM_L2L3(6) AFMM_L2L3(7) AFMM_L2L3(8)
#undef AFMM_L2L3
#undef AFMM_L2L
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_l2l(int p, bool fp32, bool parent_fp32, bool has_parent, int nsplit, const int32_t* grp, int ngrp,
                      const LevelDev& lv1, const LevelDev& lv0, const TablesDev<float>& t32,
                      const TablesDev<double>& t64, const CommonDev& cm, hipStream_t st) {
  if (ngrp == 0) return hipSuccess;
  const size_t stride = (size_t)lv0.nref * nh(p);
  if (fp32) {
    if (parent_fp32)
      return l2l_dispatch<float, float>(p, grp, ngrp, has_parent ? lv1.L32 : nullptr, lv0.rank, lv0.L32,
                                        (const float*)lv0.Lpart, nsplit, stride, t32.l2lw, cm, st);
    return l2l_dispatch<float, double>(p, grp, ngrp, has_parent ? lv1.L64 : nullptr, lv0.rank, lv0.L32,
                                       (const float*)lv0.Lpart, nsplit, stride, t32.l2lw, cm, st);
  }
  return l2l_dispatch<double, double>(p, grp, ngrp, has_parent ? lv1.L64 : nullptr, lv0.rank, lv0.L64,
                                      (const double*)lv0.Lpart, nsplit, stride, t64.l2lw, cm, st);
}

template <typename T>
static hipError_t near_dispatch(int p, int ngrp, const int32_t* grp, const LevelDev& lv1, const LevelDev& lv0,
                                const TablesDev<T>& tb, const T* Lpar, const T* part, const T* nmp, double G,
                                double h, double cself, double* phi, double* acc, hipStream_t st) {
  const int ntiles = (ngrp + 15) / 16;
  const dim3 grid(8 * ((ntiles + 7) / 8)), block(kBlock);
  switch (p) {
#define AFMM_NEAR(PP)                                                                                         \
  case PP:                                                                                                    \
    hipLaunchKernelGGL((k_near<T, PP>), grid, block, 0, st, grp, ngrp, lv1, lv0, tb.nearA, Lpar, part, nmp,  \
                       G, h, cself, phi, acc);                                                                \
    break;
    AFMM_NEAR(1) AFMM_NEAR(2) AFMM_NEAR(3) AFMM_NEAR(4) AFMM_NEAR(5) AFMM_NEAR(6) AFMM_NEAR(7) AFMM_NEAR(8)
#undef AFMM_NEAR
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_near(int p, bool fp32, int l, int l_first, const int32_t* grp, int ngrp, const LevelDev& lv1,
                       const LevelDev& lv0, const LevelDev& lvp, const TablesDev<float>& t32,
                       const TablesDev<double>& t64, const CommonDev& cm, const void* part, const void* nmp,
                       double G, double h, double cself, double* phi, double* acc, hipStream_t st) {
  (void)cm;
  (void)lvp;
  if (ngrp == 0) return hipSuccess;
  const bool has_far = (l - 1) >= l_first;
  if (fp32)
    return near_dispatch<float>(p, ngrp, grp, lv1, lv0, t32, has_far ? lv1.L32 : nullptr, (const float*)part,
                                (const float*)nmp, G, h, cself, phi, acc, st);
  return near_dispatch<double>(p, ngrp, grp, lv1, lv0, t64, has_far ? lv1.L64 : nullptr, (const double*)part,
                               (const double*)nmp, G, h, cself, phi, acc, st);
}

template <typename T>
static hipError_t near_m2p_dispatch(int p, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                                    const LevelDev& lvp, const T* Dsame, const T* S0, T* nmp, hipStream_t st) {
  const dim3 grid(ngrp), block(kBlock);
  switch (p) {
#define AFMM_NM2P(PP)                                                                                          \
  case PP:                                                                                                     \
    hipLaunchKernelGGL((k_near_m2p<T, PP>), grid, block, 0, st, grp, ngrp, lv1, lv0, lvp, Dsame, S0, nmp);     \
    break;
    AFMM_NM2P(1) AFMM_NM2P(2) AFMM_NM2P(3) AFMM_NM2P(4) AFMM_NM2P(5) AFMM_NM2P(6) AFMM_NM2P(7) AFMM_NM2P(8)
#undef AFMM_NM2P
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_near_m2p(int p, bool fp32, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                           const LevelDev& lvp, const TablesDev<float>& t32, const TablesDev<double>& t64, void* nmp,
                           hipStream_t st) {
  if (ngrp == 0) return hipSuccess;
  if (fp32) return near_m2p_dispatch<float>(p, grp, ngrp, lv1, lv0, lvp, t32.Dsame, lv0.S32, (float*)nmp, st);
  return near_m2p_dispatch<double>(p, grp, ngrp, lv1, lv0, lvp, t64.Dsame, lv0.Sc64, (double*)nmp, st);
}

}  // namespace afmm
