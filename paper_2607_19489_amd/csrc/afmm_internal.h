// Internal declarations shared by the host plan builder and the HIP kernels.
//
// Units.  Every level works in its own cell units so that FP32 coefficients
// stay O(1) at any depth:
//   S~_f[r]_a = sum_{leaves x under r} m_x ((x_x - c_r) / h_f)^a        (multipoles)
//   L~_f[r]_b = h_f^(1+|b|) d^b(phi/G) at c_r                          (local expansions)
//   phi_c = (G / h_l) phi~_c,   a_c = (G / h_l^2) a~_c                   (outputs)
// With these, every translation operator is a fixed table on unit offsets:
//   M2M  S~_a[r] = sum_o sum_{k<=a} C(a,k) d_o^(a-k) 2^-|k| S~_k[child o],  d_o = (o - 1/2)/2
//   M2L  L~_b[y] = sum_a (-1)^|a|/a! 2^|a| D~_{a+b}(R~) S~_a[s],  R~ = -2(s - F) + o_y - 1/2
//   L2L  L~_b[y] = 2^(-1-|b|) sum_g u^g/g! L~_{b+g}[F],  u = (o_y - 1/2)/2
//   M2P  phi~ = sum_a (-1)^|a|/a! 2^|a| D~_a(R~) S~_a,  a~_i = -sum_{|a|<p} (...) D~_{a+e_i} S~_a
//   L2P  phi~ = 1/2 sum_b L~_b u^b/b!,  a~_i = -1/4 sum_{b_i>0} L~_b u^(b-e_i)/(b-e_i)!
// where D~_g = d^g(-1/r) on unit offsets (Sec. 2 Eqs. eq:M2M_general, eq:M2L, eq:L2L).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <exception>
#include <memory>
#include <thread>
#include <vector>

#include "afmm.h"
#include "host_pool.h"

namespace afmm {

// Morton key of cell (x, y, z): bit b of x, y, z at bits 3b, 3b + 1, 3b + 2;
// every level of a plan is ordered by it.
inline uint64_t morton3(uint32_t x, uint32_t y, uint32_t z) {
  auto spread = [](uint64_t v) {
    v &= 0x1fffff;
    v = (v | v << 32) & 0x1f00000000ffffULL;
    v = (v | v << 16) & 0x1f0000ff0000ffULL;
    v = (v | v << 8) & 0x100f00f00f00f00fULL;
    v = (v | v << 4) & 0x10c30c30c30c30c3ULL;
    v = (v | v << 2) & 0x1249249249249249ULL;
    return v;
  };
  return spread(x) | (spread(y) << 1) | (spread(z) << 2);
}

constexpr int kMaxLevel = 21;
constexpr int kPMax = 8;
constexpr int kKMax = 165;          // C(kPMax + 3, 3)
constexpr int kNumD = 343;          // offsets d in [-3, 3]^3

__host__ __device__ constexpr int nmi(int p) { return (p + 1) * (p + 2) * (p + 3) / 6; }
// number of pairs (a, k) with k <= a componentwise and |a| <= p: C(p + 6, 6)
__host__ __device__ constexpr int nmi_entries(int p) {
  return (p + 1) * (p + 2) * (p + 3) * (p + 4) * (p + 5) * (p + 6) / 720;
}

// Position of multi-index (a, b, c) in the degree-graded order (degree, then a
// descending, then b descending).
__host__ __device__ constexpr int mi_index(int a, int b, int c) {
  return (a + b + c) * (a + b + c + 1) * (a + b + c + 2) / 6 + (b + c) * (b + c + 1) / 2 + c;
}

// Harmonic form.  The derivatives of 1/r obey D_{g+2ez} = -D_{g+2ex} - D_{g+2ey},
// so of the K = C(p+3, 3) Cartesian coefficients of an expansion only the
// (p + 1)^2 with c <= 1 (multi-index (a, b, c)) are independent in a sum with
// them: the coefficients with c >= 2 are folded onto those of the same order
// before the sum (source copies), and the local expansions that M2L forms obey
// the same relation, so M2L computes only those with c <= 1 and the others
// follow (k_l2l).  Exact at every truncation: folding keeps the order, and the
// products of M2L and M2P shrink from 924 to 532 and from 84 + 3 56 to 49 + 3 36
// terms at p = 6.  Position of (a, b, c), c <= 1, in the degree-graded folded order:
__host__ __device__ constexpr int nh(int p) { return (p + 1) * (p + 1); }
__host__ __device__ constexpr int h_index(int a, int b, int c) { return (a + b + c) * (a + b + c) + c * (a + b + c + 1) + b; }
__host__ __device__ constexpr int h_deg(int h) {
  int n = 0;
  while ((n + 1) * (n + 1) <= h) ++n;
  return n;
}
// position in the full order of folded coefficient h
__host__ __device__ constexpr int h_full(int h) {
  const int n = h_deg(h), r = h - n * n, c = r > n ? 1 : 0, b = r - c * (n + 1);
  return mi_index(n - b - c, b, c);
}

// parities of folded coefficient h (bit i: axis i)
__host__ __device__ inline int h_parity(int h) {
  int n = 0;
  while ((n + 1) * (n + 1) <= h) ++n;
  const int r = h - n * n, c = r > n ? 1 : 0, b = r - c * (n + 1);
  return ((n - b - c) & 1) | (b & 1) << 1 | c << 2;
}

// Layout of the scaled source copies (S32 / Sc64): the KH = nh(p) folded
// coefficients in NP passes of 16 blocks of CP values, [pass][block][CP], every
// block holding coefficients of one parity class (the parities of a, b, c), so
// that the reflections of a block's values are one sign per lane (M2P, M2L).
// Lane q of 16 loads block q of a row as one vector of CP values (at most 16
// bytes); unused slots are 0.  The eight classes need no more than 16 blocks
// with 1, 1, 1, 2, 3, 4, 6, 6 values for p = 1..8 (49 of 64 slots hold a
// coefficient at p = 6).  Behind the nref rows comes one row of zeros, read for
// a missing or leaf source.
constexpr int kSymBlocks = 16;
__host__ __device__ constexpr int sym_cpl(int p) { return p <= 3 ? 1 : p <= 6 ? p - 2 : 6; }
__host__ __device__ constexpr int sym_cp(int p, int bytes) {
  return bytes == 4 ? (sym_cpl(p) <= 4 ? sym_cpl(p) : 3) : (sym_cpl(p) == 1 ? 1 : 2);
}
__host__ __device__ constexpr int sym_np(int p, int bytes) { return (sym_cpl(p) + sym_cp(p, bytes) - 1) / sym_cp(p, bytes); }
__host__ __device__ constexpr int src_row(int p, int bytes) { return sym_np(p, bytes) * kSymBlocks * sym_cp(p, bytes); }

template <int P, int BYTES>
struct SymLayout {
  static constexpr int CP = sym_cp(P, BYTES), NP = sym_np(P, BYTES), ROW = src_row(P, BYTES);
  int pos[nh(P)];             // slot of folded coefficient h
  int coef[ROW];              // coefficient of a slot, or -1
  int par[kSymBlocks];        // parity class of a block (bit i: axis i odd)
  constexpr SymLayout() : pos(), coef(), par() {
    for (int i = 0; i < ROW; ++i) coef[i] = -1;
    int blk = 0;
    for (int c = 0; c < 8; ++c) {
      int j = 0;
      for (int n = 0; n <= P; ++n)
        for (int z = 0; z <= (n > 0 ? 1 : 0); ++z)
          for (int b = 0; b <= n - z; ++b) {
            const int a = n - b - z;
            if (((a & 1) | (b & 1) << 1 | (z & 1) << 2) != c) continue;
            const int q = blk + j / (NP * CP), e = j % (NP * CP);
            const int at = (e / CP * kSymBlocks + q) * CP + e % CP;
            pos[h_index(a, b, z)] = at;
            coef[at] = h_index(a, b, z);
            par[q] = c;
            ++j;
          }
      blk += (j + NP * CP - 1) / (NP * CP);
    }
  }
};

// Rows of the adjoint's local-expansion bars: the KH folded coefficients in the order in
// which its kernel reads the B operand straight into registers.  Lane group g
// (lane >> 4) of a 16x16x4 step kb holds coefficient k = 4 kb + g.  A lane group
// needs STP steps (STP = ceil(KH/4) rounded up to whole 16-byte vectors of VW =
// 16/bytes values); its vector j holds steps VW j .. VW j + VW - 1.  The row
// stores the vectors j-major: vector j of lane group g at (4 j + g) VW, so one
// 16-byte load per lane (vector j for all 4 lane groups of a source) reads 64
// contiguous bytes of each source row.  Coefficient k therefore sits at
// ((k >> 2) / VW) 4 VW + (k & 3) VW + (k >> 2) % VW; unused slots are 0.
__host__ __device__ constexpr int folded_stp(int p, int bytes) {
  return (((nh(p) + 3) / 4) + (16 / bytes) - 1) / (16 / bytes) * (16 / bytes);
}
__host__ __device__ constexpr int folded_row(int p, int bytes) { return 4 * folded_stp(p, bytes); }
__host__ __device__ constexpr int src_pos(int k, int bytes) {
  return ((k >> 2) / (16 / bytes)) * 4 * (16 / bytes) + (k & 3) * (16 / bytes) + (k >> 2) % (16 / bytes);
}
// element offset of vector j of lane group g in such a row
__host__ __device__ constexpr int src_vec(int j, int g, int bytes) { return (4 * j + g) * (16 / bytes); }

// The 189 source offsets of a group (d in [-2, 3] on each axis, mirrored where the
// group's octant bit is set, less the 27 near ones) as 56 orbits under the
// reflections of the axes: on each axis the offsets are {0}, {-1, 1}, {-2, 2} and
// {3}.  All sources of an orbit are in one octant of their fathers: the group's,
// with the bits of m flipped, m the axes with an odd offset.  Per m there is one
// orbit for every set PT of reflected axes but PT = m (the near offsets): offset
// 1 or 2 on a reflected axis, 3 or 0 on the others as m is set or not.  Orbit
// w = 7 m + j takes the j-th set of sym_axes(0..7) without m; bit b of a source's
// index is set where its offset on the b-th axis of PT is negative.
constexpr int kSymOrbits = 56;
__host__ __device__ constexpr int sym_axes(int t) { return (0x01243567 >> (4 * t)) & 7; }
__host__ __device__ constexpr int sym_bits(int pt) { return (pt & 1) + ((pt >> 1) & 1) + ((pt >> 2) & 1); }
// position t of orbit (m, j)'s set
__host__ __device__ constexpr int sym_set(int m, int j) {
  const int t = sym_axes(m);  // the order is its own inverse: m's position in it
  return j < t ? j : j + 1;
}

// Variants of an orbit's operator (M2L): one per set of the axes, among those of m
// that it does not reflect, on which the group's class has its offset 3 on the
// negative side; 1, 2, 4 or 8 per orbit, 117 in all.
constexpr int kSymVariants = 117;
// E rows of a variant: character x at x * sym_es(p), coefficients g < K then zeros,
// one zero slot at 8 * sym_es(p), zeros to whole 16-byte vectors.  The stride is
// the one with the fewest LDS bank conflicts of the A operand's gathers (counted
// for 4- and 8-byte values; 2.9 passes of 64 lanes at p = 6, 3.8 without padding).
__host__ __device__ constexpr int sym_es(int p) {
  return p <= 5 ? 80 : p == 6 ? 96 : p == 7 ? 144 : 176;
}
__host__ __device__ constexpr int sym_elen(int p, int bytes) {
  return (8 * sym_es(p) + 1 + 16 / bytes - 1) / (16 / bytes) * (16 / bytes);
}
// M2L sums tap by tap up to p = 4 and by orbits from p = 5.  An orbit's loads,
// butterflies and barrier cost the same at any order, its products grow with p^4:
// 64^3 + 1 level in FP32, taps / orbits 77 / 90 us at p = 4, 105 / 103 at p = 5,
// 150 / 126 at p = 6, 329 / 211 at p = 8 (FP64: 115 / 131, 167 / 167, 277 / 203).  The
// line is one of orders alone: a batch and its members' own plans, of other sizes,
// give the same bits at equal splits.
__host__ __device__ constexpr bool m2l_by_taps(int p) { return p <= 4; }
// Columns of an M2L tile; by orbits, two tiles of 16 per wave share the A operand
// where both sets of U fit the LDS.
constexpr int kM2LBlock = 512;
__host__ __device__ constexpr int m2l_cols(int p, int bytes) {
  return !m2l_by_taps(p) && bytes == 4 && p <= 6 ? 32 : 16;
}

// D~ rows of one source offset in the layout the MFMA kernels stage in LDS:
// row o (child octant) at o * dstage_ks(p), coefficients g < K then zeros up
// to the stride, one zero slot at 8 * dstage_ks(p), zero padding to whole
// 16-byte vectors for every lane of a wave.  Copied to LDS as is.  The row
// stride is chosen per order (at least K rounded up to 4, same padded length)
// to spread the A-operand gathers (8 rows x derivative-shifted
// coefficient indices per lane) over the LDS banks; chosen by counting bank
// conflicts of those offset tables for 32- and 64-bank LDS models.
__host__ __device__ constexpr int dstage_ks(int p) {
  return p == 1 ? 6 : p == 2 ? 30 : p == 3 ? 28 : p == 4 ? 52 : p == 5 ? 57 : p == 6 ? 93 : p == 7 ? 121 : 185;
}
__host__ __device__ constexpr int dstage_len(int p, int bytes) {
  return (8 * dstage_ks(p) + 1 + 64 * (16 / bytes) - 1) / (64 * (16 / bytes)) * (64 * (16 / bytes));
}

// Near field of one group as a fixed linear map (Sec. 3.2, Alg. 4): the 8
// targets (rows c * 8 + o, c = phi, ax, ay, az) take P2P from the 216 children
// of the father's 27 neighbours (columns 8 e + o'), P2P from the 27
// neighbours themselves when they are leaves one level coarser (columns
// 216 + e), and L2P from the father's local expansion (columns 243 + b).
// Columns are padded to whole 16-byte vectors of MFMA steps for both
// precisions; the operator is stored per lane of the 16x16x4 A operand:
// element [t][kb / VW][lane][kb % VW] is row 16 t + (lane & 15), column
// 4 kb + (lane >> 4), VW = 16 / bytes.
constexpr int kNearLeafCols = 216;
constexpr int kNearCoarseCols = 27;
__host__ __device__ constexpr int near_cols(int p) { return (kNearLeafCols + kNearCoarseCols + nmi(p) + 15) / 16 * 16; }
__host__ __device__ constexpr int near_ksteps(int p) { return near_cols(p) / 4; }

// Interaction-list taps per octant class: the children of the father's 27
// neighbours (216) less the cell's own 27 neighbours.
constexpr int kTapsPerClass = 189;

// Work items of one launch split into 8 contiguous ranges, one per XCD (the
// hardware deals workgroups to the XCDs round-robin): workgroup b runs item
// start[b % 8] + b / 8 if that is below start[b % 8 + 1].  Ranges of equal
// estimated work rather than equal length keep every XCD busy when the work
// per item varies; each XCD still reads a contiguous run of tiles.
struct XcdRanges {
  int32_t start[9] = {};
  int32_t grid() const {
    int32_t m = 0;
    for (int x = 0; x < 8; ++x) m = start[x + 1] - start[x] > m ? start[x + 1] - start[x] : m;
    return 8 * m;
  }
};

// Per-level device view.  Level l holds the children of the refined cells of
// level l - 1 in Morton order, so cell index c has father refined rank c >> 3
// and octant c & 7 (o = ox + 2 oy + 4 oz), and refined rank r owns children
// 8r .. 8r+7.  Neighbour index e = (ex+1) + 3(ey+1) + 9(ez+1).
struct LevelDev {
  int32_t n = 0;             // cells
  int32_t nref = 0;          // refined cells
  const int32_t* rank = nullptr;     // [n] refined rank or -1 (leaf)
  const int32_t* slot = nullptr;     // [n] caller slot (flat index) or -1 (cells above levelmin)
  const int32_t* refcell = nullptr;  // [nref] cell index of refined rank r
  const int32_t* nbr = nullptr;      // [nref][27] neighbour cell index at this level, -1 outside box
  double* mass = nullptr;            // [n] leaf masses of this solve (0 for refined cells)
  double* S64 = nullptr;             // [nref][K] multipoles (FP64), used by the upward pass
  float* S32 = nullptr;              // [nref][src_row(p, 4)] source copy (-1)^|a|/a! 2^|a| S~_a, folded, FP32
                                     // (mixed form), in the layout above
  double* Sc64 = nullptr;            // [nref][src_row(p, 8)] same source copy in FP64
  double* L64 = nullptr;             // [nref][K] local expansions (FP64 levels)
  float* L32 = nullptr;              // [nref][K] local expansions (FP32 levels)
  void* part = nullptr;              // [npart][nref][32] intermediate-field partials of the leaf children (T of the
                                     // leaf level), one set per M2P tap range
  int32_t npart = 0;
  size_t part_bytes = 0, Lpart_bytes = 0;
  void* Lpart = nullptr;             // [nsplit][nref][nh(p)] M2L tap-range partial sums (T of the level), if split
  // adjoint pass (FP64, allocated by the first adjoint call)
  double* tbar = nullptr;            // [n][4] unit-form bars of the target leaves (phi, ax, ay, az)
  double* mbar = nullptr;            // [n] mass bars of the leaves
  double* sbar = nullptr;            // [nref][K] source-copy bar, then multipole bar
  double* lbar = nullptr;            // [nref][K] local-expansion bar
  void* tbT = nullptr;               // [nref][32] target bars of the leaf children, B of the transposed M2P (T)
  void* lbarT = nullptr;             // [nref][folded_row] local-expansion bar, B of the transposed M2L (T, lane-group layout)
};

template <typename T>
struct TablesDev {
  const T* Dstage = nullptr;  // [kNumD][dstage_len(p, sizeof(T))] D~ at R~ = -2d + o - 1/2, 8 rows per d,
                              // in the LDS stage layout of the MFMA kernels
  const T* Dsame = nullptr;   // [kNumD][K]      D~ at integer R~ in [-3,3]^3
  const T* cfacn = nullptr;   // [K] 2^-|a| (FP64): same-level M2P from the source copies, transposed
  const T* l2lw = nullptr;    // [8][p+1][K] L2L weights 2^(-1-|b|) u^g/g! per child octant and |b|
  const T* l2p = nullptr;     // [8][4][K] L2P weights (phi, ax, ay, az) per child octant
  const T* nearA = nullptr;   // [2][near_ksteps / VW][64][VW] near-field operator, MFMA A layout
  const T* symE = nullptr;    // [kSymVariants][sym_elen] E rows of the orbits (M2L)
  const T* symA = nullptr;    // [8 m][NP][7][8][64][CP] M2P operator per orbit, pass and character (SymLayout)
  const T* adjNearA = nullptr;  // [216][64] transposed same-level near field (adjoint), MFMA A layout
};

struct CommonDev {
  const int16_t* sumidx = nullptr;  // [K][K] index of a + b (or -1 when |a|+|b| > p)
  const int16_t* up = nullptr;      // [K][3] index of a + e_i (or -1 when |a| = p)
  const int8_t* mi = nullptr;       // [K][4] (a, b, c, |a|)
  const double* binom = nullptr;    // [(kPMax+1)^2] binomial coefficients C(n, k) at n*(kPMax+1)+k
  const double* fold_u = nullptr;   // weights of the fold lists without the source copies' factors
  const double* cfac2 = nullptr;    // [K] (-1)^|a|/a! 2^|a| (FP64), the factors of the source copies
  const int32_t* fold_start = nullptr;  // [nh + 1] entry range of each folded source coefficient
  const int16_t* fold_list = nullptr;   // entries: coefficient a
  const double* fold_w = nullptr;       // weights cfac2_a times the signed binomial of the fold
  const double* fold_p2m = nullptr;     // [nh] the same applied to the k = 0 entry of each a's M2M list (leaf children)
  const int32_t* m2m_start = nullptr;  // [K+1] M2M entry range of each coefficient a
  const int32_t* m2m_list = nullptr;   // entries: k | parity(a-k) << 12
  const double* m2m_w = nullptr;       // entry weights C(a,k) 4^-|a-k| 2^-|k|
  const int32_t* m2mT_start = nullptr; // [K+1] the same entries grouped by k (adjoint)
  const int32_t* m2mT_list = nullptr;  // entries: a | parity(a-k) << 12
  const double* m2mT_w = nullptr;
  const int32_t* tapsT = nullptr;      // [8][189] per source octant: e | oF << 5 | d_index << 8 (adjoint)
  const int16_t* adj_m2p_off = nullptr; // [RT * 8][64] A offsets of the transposed M2P
  const int16_t* adj_m2l_off = nullptr; // [steps][64] A offsets (within one D~ row) of the transposed M2L
  const int32_t* l2lT_start = nullptr;  // [K+1] transposed L2L pairs of each coefficient c
  const int32_t* l2lT_list = nullptr;   // b | (c - b) << 8 | |b| << 16 | parity(c - b) << 24
  const double* l2lT_w = nullptr;       // [entries] weight 2^(-1-|b|) u_7^(c-b)/(c-b)! of child 7 (u_7 = +1/4)
};

// Group tiles of the MFMA kernels: NC refined ranks per tile (one parity class,
// -1 padded), tiles of the 8 classes interleaved.
struct MfmaTiles {
  const int32_t* tiles = nullptr;
  int ntiles = 0;
  int nc = 0;
};

struct MfmaTables {
  const int8_t* symtaps = nullptr;    // [8][56][8] per parity class and orbit: its sources' fathers (neighbour e)
  const int* symvar = nullptr;        // [8][56] per parity class and orbit: its variant
  const int32_t* taps = nullptr;      // [8][189] per parity class: e | o' << 5 | d_index << 8
  const int16_t* m2l_off = nullptr;   // places of M2L's A operand: [steps][64] in D~ rows (taps), or
                                      // [8][steps][64] in a variant's E rows, per character (orbits)
};

// Launchers (afmm_kernels.hip).  All return hipGetLastError() of the launch.
// Leaf masses of one level from the caller's slot array; with `snap`, every
// cell's slot value is also copied there (the adaptive-time-step snapshot).
hipError_t launch_gather_mass(const LevelDev& lv, const double* m_src, double* snap, hipStream_t st);
// Drifted masses of a solve with stale trees: out[s] = m[s] + dt * rate[s] for
// the slots [off[i], off[i + 1]) of AMR level i (levels with dt = 0 copied)
struct DriftLevels {
  int n = 0;
  int64_t off[kMaxLevel + 1] = {};
  double dt[kMaxLevel] = {};
};
hipError_t launch_drift(const DriftLevels& d, const double* m, const double* rate, double* out, int64_t nslots,
                        hipStream_t st);
hipError_t launch_copy_slots(const int32_t* slots, int64_t n, const double* src, double* dst,
                             hipStream_t st);
// Batches: forest slot <-> caller arrays.  leafslot/leafhier list every leaf of
// the forest with its hierarchy; base[h] is the hierarchy's first forest slot.
hipError_t launch_batch_in(int64_t nleaf, const int32_t* leafslot, const int32_t* leafhier, const int64_t* base,
                           const double* const* mass, double* m_forest, hipStream_t st);
hipError_t launch_batch_out(int64_t nleaf, const int32_t* leafslot, const int32_t* leafhier, const int64_t* base,
                            const double* phi_forest, const double* acc_forest, double* const* phi,
                            double* const* acc, hipStream_t st);
// Adjoint pass (afmm_adjoint.hip).
hipError_t launch_adj_init(const LevelDev& lv, int target, const double* phib, const double* accb, double sp,
                           double sa, hipStream_t st);
hipError_t launch_adj_zero(double* p, size_t n, hipStream_t st);
// Adjoint near field of level l: the same-level P2P^T of the leaf groups as
// one MFMA product (targets_here only), the coarse and nearest P2P^T of the
// groups in vgrp (those with a leaf neighbour one level coarser or a refined
// near candidate), the near M2P^T of refgrp.
hipError_t launch_adj_near(int p, const int32_t* leafgrp, int nleafgrp, const int32_t* vgrp, int nvgrp,
                           const int32_t* refgrp, int nrefgrp, const LevelDev& lv1, const LevelDev& lv0,
                           const LevelDev& lvp, int targets_here, const TablesDev<double>& t64, const CommonDev& cm,
                           hipStream_t st);
hipError_t launch_adj_l2p(int p, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                          const TablesDev<double>& t64, const CommonDev& cm, hipStream_t st);
// MFMA forms: tiles of 16 source cells (records: target level, 16 cells); with
// nsplit > 1 the 189 taps of a tile are split over blocks writing partial sets
// into `part` ([nsplit][ntiles * 16][nh(p)] FP64), summed in order afterwards.
// Periodic boxes: the level-2 far operator table ([8][kNumD][K] in level-2
// units, cached per order) and its kernel (writes L of the 64 level-2 cells).
std::shared_ptr<const std::vector<double>> periodic_far_table(int p);
hipError_t launch_periodic_far(int p, const LevelDev& lv2, const double* T, const double* cf, const CommonDev& cm,
                               hipStream_t st);
// its transpose: level-2 multipole bars from the level-2 local-expansion bars
hipError_t launch_adj_periodic_far(int p, const LevelDev& lv2, const double* T, const double* cf,
                                   const CommonDev& cm, hipStream_t st);
hipError_t launch_adj_m2p_mfma(int p, bool fp32, const int32_t* tiles, int ntiles, int nsplit, const XcdRanges& xr,
                               const uint8_t* live, double* part,
                               const int32_t* tapsT, const int16_t* aoff, const LevelDev& lvp, const LevelDev& lvs,
                               const LevelDev& lvt, const TablesDev<float>& t32, const TablesDev<double>& t64,
                               const CommonDev& cm, hipStream_t st);
hipError_t launch_adj_m2l_mfma(int p, bool fp32, const int32_t* tiles, int ntiles, int nsplit, const XcdRanges& xr,
                               const uint8_t* live, double* part,
                               const int32_t* tapsT, const int16_t* aoff, const LevelDev& lvp, const LevelDev& lvs,
                               const LevelDev& lvt, const TablesDev<float>& t32, const TablesDev<double>& t64,
                               const CommonDev& cm, hipStream_t st);
hipError_t launch_adj_l2l(int p, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                          const TablesDev<double>& t64, const CommonDev& cm, hipStream_t st);
hipError_t launch_adj_down(int p, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                           int has_parent, const CommonDev& cm, hipStream_t st);
// Mass bars to the caller's slots; cself (the self-potential constant, 0 when
// off) adds the transpose of the self term -cself m of the unit-form potential.
hipError_t launch_adj_out(int p, const LevelDev& lv1, const LevelDev& lv0, int has_parent, int rebuilt,
                          double cself, const CommonDev& cm, double* mbar_out, hipStream_t st);
// Upward pass of FMM level f: the refined cells whose children are all leaves
// (list leaf, P2M only) and the others (list mix, M2M of refined children).
hipError_t launch_upward(int p, const int32_t* leaf, int nleaf, const int32_t* mix, int nmix, const LevelDev& lv,
                         const LevelDev& lvc, const CommonDev& cm, hipStream_t st);
// M2P tiles: quads of groups per wave (4 waves), groups per tile, and the most
// distinct fathers of sources of one tile.  Two blocks share a CU's LDS, which
// holds one octant's rows of those fathers in vectors of 4 values (of 8 bytes or
// less for the low orders): 200 fathers cover 48 groups of a filled region, 240
// 64 groups.
__host__ __device__ constexpr int m2p_vec(int p, int bytes) { return sym_cp(p, bytes) == 3 ? 4 : sym_cp(p, bytes); }
__host__ __device__ constexpr int m2p_quads(int p, int bytes) { return m2p_vec(p, bytes) * bytes == 16 ? 3 : 4; }
__host__ __device__ constexpr int m2p_cols(int p, int bytes) { return 16 * m2p_quads(p, bytes); }
__host__ __device__ constexpr int m2p_fathers(int p, int bytes) { return m2p_quads(p, bytes) == 3 ? 200 : 240; }
// MFMA launches over a contiguous range [t0, t0 + n) of tile records; each
// record is (target level, NC groups); a direct M2P tile's has its quads per wave
// above the level's 8 bits.  lvs is the device array of LevelDev.
hipError_t launch_m2l(int p, bool fp32, const MfmaTiles& mt, int t0, int n, int nsplit, const MfmaTables& tabs,
                           const LevelDev* lvs, const TablesDev<float>& t32, const TablesDev<double>& t64,
                           hipStream_t st);
hipError_t launch_l2l(int p, bool fp32, bool parent_fp32, bool has_parent, int nsplit, const int32_t* grp, int ngrp,
                      const LevelDev& lv1, const LevelDev& lv0, const TablesDev<float>& t32,
                      const TablesDev<double>& t64, const CommonDev& cm, hipStream_t st);
hipError_t launch_m2p(int p, bool fp32, const MfmaTiles& mt, int t0, int n, int nsplit,
                      const MfmaTables& tabs, const LevelDev* lvs, const TablesDev<float>& t32,
                      const TablesDev<double>& t64, hipStream_t st);
// cself: the self-potential constant (AFMM_SELF_POTENTIAL), 0 when off.
hipError_t launch_near(int p, bool fp32, int l, int l_first, const int32_t* grp, int ngrp, const LevelDev& lv1,
                       const LevelDev& lv0, const LevelDev& lvp, const TablesDev<float>& t32,
                       const TablesDev<double>& t64, const CommonDev& cm, const void* part, const void* nmp,
                       double G, double h, double cself, double* phi, double* acc, hipStream_t st);
// Near-field M2P from the refined level-l cells among the near candidates of
// the groups `grp` (those that have any): partial [nref(l-1)][c * 8 + o].
hipError_t launch_near_m2p(int p, bool fp32, const int32_t* grp, int ngrp, const LevelDev& lv1, const LevelDev& lv0,
                           const LevelDev& lvp, const TablesDev<float>& t32, const TablesDev<double>& t64, void* nmp,
                           hipStream_t st);

}  // namespace afmm
