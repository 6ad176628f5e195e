// fmm.h -- 3D Laplace FMM for block mode: octree construction, upward and
// downward passes as data-parallel kernels, and the cell-pair work that the
// dual-tree traversal tasks run (GTaP Sec. 6.4.1).
//
// Conventions (the paper names the phases only):
//   * root cube [-2^7, 2^7)^3; grid coordinate floor((x + 2^7) * 2^13) in
//     [0, 2^21); 63-bit Morton key (bit 3k+2: x, 3k+1: y, 3k: z); points sorted
//     by (key, index);
//   * a cell splits iff it holds more than leaf_max points below level 21;
//     only non-empty children; cells numbered level by level in Morton order;
//   * MAC theta = ta/tb on doubled integer centres:
//     accept iff 3 tb^2 (w_A + w_B)^2 < ta^2 |C2_A - C2_B|^2;
//   * Cartesian Taylor expansions of 1/|x - y| of total degree <= 6:
//     moments Q_b = sum q (y - c_B)^b, locals
//     L_a = sum_b C(a+b, a) (-1)^|b| T_{a+b}(c_A - c_B) Q_b, where T_g are the
//     Taylor coefficients of 1/|d + h| from the Coulomb three-term recurrence;
//   * M2L runs on reduced sets.  With T'_g = g! T_g, Q'_b = (-1)^|b| Q_b / b! and
//     L'_a = a! L_a it is L'_a = sum_b T'_{a+b} Q'_b, and since 1/r is harmonic,
//     T'_{g+2ez} = -T'_{g+2ex} - T'_{g+2ey}.  So moments with b_z >= 2 fold into
//     those with b_z <= 1 (49 of 84), locals with a_z >= 2 follow from the
//     others (both exactly, degree by degree), and the contraction has 532
//     terms on 64 derivatives (g_z <= 2) instead of 924 on 84.
#pragma once
#include "layout.h"
#include "wave.h"

namespace gtap {
namespace fmm {

constexpr int kP = 6;                                          // expansion order
constexpr int kNc = (kP + 1) * (kP + 2) * (kP + 3) / 6;        // 84 coefficients
constexpr int kBits = 21;                                      // tree depth limit
constexpr int kE = 7;                                          // root half-width 2^7
constexpr int kGrid = kBits - 1 - kE;                          // 2^13 grid units per unit length
constexpr int kCellInts = 8;                                   // level ax ay az begin end child0 nchild

// Number of coefficients of total degree <= d.
constexpr int ncoef(int d) { return (d + 1) * (d + 2) * (d + 3) / 6; }
constexpr int kNr = (kP + 1) * (kP + 1);  // 49 reduced coefficients (z exponent <= 1), 2 d + 1 of degree d
constexpr int nred(int d) { return (d + 1) * (d + 1); }  // of degree <= d
// Doubles between two cells' reduced moments: degrees <= 4 (25) from 0, degrees
// 5 and 6 (24) from 26 -- two halves of thirteen 16-byte units.
constexpr int kQrStride = 52;
constexpr int qr_at(int r) { return r < nred(4) ? r : r + 1; }
constexpr int kNg = kNr + (kP - 1) * kP / 2;  // 64 derivatives with z exponent <= 2: the reduced ones, then z = 2
constexpr int kM2LTerms = 532;  // pairs (a, b) of reduced coefficients with |a| + |b| <= 6

// Multi-index tables, generated at compile time.  Coefficients are ordered by
// total degree, then by descending x and y exponents.
struct Tables {
  uint8_t e[kNc][3];                     // exponents of coefficient t
  uint8_t idx[kP + 1][kP + 1][kP + 1];   // inverse of e
  uint8_t deg[kNc];
  uint8_t dm1[kNc][3];                   // index of g - e_i (0xFF if g_i == 0)
  uint8_t red[kNr];                      // coefficient of reduced index r
  uint8_t red_of[kNc];                   // inverse (0xFF: z exponent >= 2)
  uint8_t g_of[kP + 1][kP + 1][3];       // index of derivative (x, y, z <= 2) among the 64
  uint8_t ge[kNg][3];                    // its exponents
  uint16_t m2l_first[kNr + 1];           // terms of reduced target a: [m2l_first[a], m2l_first[a+1])
  uint8_t m2l_b[kM2LTerms];              // reduced source moment b
  uint8_t m2l_g[kM2LTerms];              // derivative a + b
  double fact[kNc];                      // e_x! e_y! e_z!
  double binom[2 * kP + 1][2 * kP + 1];
};

constexpr Tables make_tables() {
  Tables T{};
  for (int n = 0; n <= 2 * kP; ++n) {
    T.binom[n][0] = 1.0;
    for (int k = 1; k <= n; ++k) T.binom[n][k] = T.binom[n - 1][k - 1] + (k < n ? T.binom[n - 1][k] : 0.0);
  }
  int t = 0;
  for (int d = 0; d <= kP; ++d)
    for (int i = d; i >= 0; --i)
      for (int j = d - i; j >= 0; --j) {
        const int k = d - i - j;
        T.e[t][0] = static_cast<uint8_t>(i);
        T.e[t][1] = static_cast<uint8_t>(j);
        T.e[t][2] = static_cast<uint8_t>(k);
        T.idx[i][j][k] = static_cast<uint8_t>(t);
        T.deg[t] = static_cast<uint8_t>(d);
        ++t;
      }
  for (int s = 0; s < kNc; ++s)
    for (int i = 0; i < 3; ++i) {
      int g[3] = {T.e[s][0], T.e[s][1], T.e[s][2]};
      T.dm1[s][i] = 0xFF;
      if (g[i] >= 1) {
        g[i] -= 1;
        T.dm1[s][i] = T.idx[g[0]][g[1]][g[2]];
      }
    }
  int r = 0;
  for (int s = 0; s < kNc; ++s) {
    double v = 1.0;
    for (int i = 0; i < 3; ++i)
      for (int k = 2; k <= T.e[s][i]; ++k) v *= k;
    T.fact[s] = v;
    T.red_of[s] = 0xFF;
    if (T.e[s][2] <= 1) {
      T.red[r] = static_cast<uint8_t>(s);
      T.red_of[s] = static_cast<uint8_t>(r);
      T.g_of[T.e[s][0]][T.e[s][1]][T.e[s][2]] = static_cast<uint8_t>(r);
      for (int i = 0; i < 3; ++i) T.ge[r][i] = T.e[s][i];
      ++r;
    }
  }
  for (int s = 0; s < kNc; ++s)
    if (T.e[s][2] == 2) {
      T.g_of[T.e[s][0]][T.e[s][1]][2] = static_cast<uint8_t>(r);
      for (int i = 0; i < 3; ++i) T.ge[r][i] = T.e[s][i];
      ++r;
    }
  int m = 0;
  for (int a = 0; a < kNr; ++a) {
    T.m2l_first[a] = static_cast<uint16_t>(m);
    const int ta = T.red[a];
    for (int b = 0; b < nred(kP - T.deg[ta]); ++b) {
      const int tb = T.red[b];
      T.m2l_b[m] = static_cast<uint8_t>(b);
      T.m2l_g[m] = T.g_of[T.e[ta][0] + T.e[tb][0]][T.e[ta][1] + T.e[tb][1]][T.e[ta][2] + T.e[tb][2]];
      ++m;
    }
  }
  T.m2l_first[kNr] = static_cast<uint16_t>(m);
  return T;
}

__constant__ const Tables kTab = make_tables();
static_assert(make_tables().m2l_first[kNr] == kM2LTerms, "M2L term count");

// Per-job device descriptor of an FMM traversal.
struct FmmDesc {
  const int32_t *cell;     // [ncells][kCellInts]
  const double *Qr;        // [ncells][kQrStride] reduced moments
  double *Lr;              // [ncells][kNr] reduced local coefficients (block mode accumulates them)
  const double *px, *py, *pz, *pq;  // points in sorted order
  double *phi;             // potentials in sorted order (accumulated)
  int64_t ta, tb;          // MAC theta = ta / tb
  uint64_t m2l_pairs, p2p_pairs, m2l_hash, p2p_hash, p2p_inter, coincident;
  // interaction lists (list-building traversals): (target << 32 | source)
  // pairs, appended at m2l_n / p2p_n, which keep counting past the capacity
  uint64_t *m2l_list, *p2p_list;
  uint64_t m2l_cap, p2p_cap;
  uint64_t m2l_n, p2p_n;
  uint32_t ncells;         // a list slot holding target ncells is a gap (see list chunks)
  uint32_t pad_;
};

GTAP_DEV double cell_centre(int32_t anchor, int32_t level) {
  const int64_t w = static_cast<int64_t>(1) << (kBits - level);
  const int64_t c2 = 2 * static_cast<int64_t>(anchor) + w;
  return -static_cast<double>(1 << kE) + static_cast<double>(c2) * (1.0 / static_cast<double>(1 << (kGrid + 1)));
}

GTAP_DEV bool mac_accept(const int32_t *A, const int32_t *B, int64_t ta, int64_t tb) {
  const int64_t wa = static_cast<int64_t>(1) << (kBits - A[0]), wb = static_cast<int64_t>(1) << (kBits - B[0]);
  const int64_t dx = (2 * static_cast<int64_t>(A[1]) + wa) - (2 * static_cast<int64_t>(B[1]) + wb);
  const int64_t dy = (2 * static_cast<int64_t>(A[2]) + wa) - (2 * static_cast<int64_t>(B[2]) + wb);
  const int64_t dz = (2 * static_cast<int64_t>(A[3]) + wa) - (2 * static_cast<int64_t>(B[3]) + wb);
  const __int128 lhs = static_cast<__int128>(3 * tb * tb) * static_cast<__int128>((wa + wb) * (wa + wb));
  const __int128 rhs = static_cast<__int128>(ta * ta) * static_cast<__int128>(dx * dx + dy * dy + dz * dz);
  return lhs < rhs;
}

GTAP_DEV uint64_t pair_hash(uint32_t a, uint32_t b) {
  uint64_t z = (static_cast<uint64_t>(a) << 32) | b;
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ---- tree construction ------------------------------------------------------
GTAP_DEV uint64_t spread3(uint64_t v) {
  v &= 0x1FFFFFull;
  v = (v | (v << 32)) & 0x1F00000000FFFFull;
  v = (v | (v << 16)) & 0x1F0000FF0000FFull;
  v = (v | (v << 8)) & 0x100F00F00F00F00Full;
  v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

GTAP_DEV int64_t grid_coord(double x) {
  const double shifted = __dadd_rn(x, static_cast<double>(1 << kE));
  return static_cast<int64_t>(floor(__dmul_rn(shifted, static_cast<double>(1 << kGrid))));
}

__global__ void k_keys(int32_t n, const double *x, const double *y, const double *z, uint64_t *keys,
                       int32_t *idx, int32_t *bad) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t gx = grid_coord(x[i]), gy = grid_coord(y[i]), gz = grid_coord(z[i]);
  const int64_t lim = static_cast<int64_t>(1) << kBits;
  if (gx < 0 || gy < 0 || gz < 0 || gx >= lim || gy >= lim || gz >= lim) {
    atomicAdd(bad, 1);
    keys[i] = 0;
  } else {
    keys[i] = (spread3(static_cast<uint64_t>(gx)) << 2) | (spread3(static_cast<uint64_t>(gy)) << 1) |
              spread3(static_cast<uint64_t>(gz));
  }
  idx[i] = i;
}

__global__ void k_gather(int32_t n, const int32_t *perm, const double *x, const double *y, const double *z,
                         const double *q, double *px, double *py, double *pz, double *pq, double *phi) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t i = perm[k];
  px[k] = x[i];
  py[k] = y[i];
  pz[k] = z[i];
  pq[k] = q[i];
  phi[k] = 0.0;
}

__global__ void k_root(int32_t *cell, int32_t *parent, int32_t n) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const int32_t r[kCellInts] = {0, 0, 0, 0, 0, n, 0, 0};
    for (int i = 0; i < kCellInts; ++i) cell[i] = r[i];
    parent[0] = -1;
  }
}

// Cells [lo, hi) of one level: octant boundaries of each splitting cell by
// binary search in its sorted key range, and the number of non-empty children;
// *nsplit counts the cells that split.
__global__ void k_level_count(int32_t *cell, int32_t lo, int32_t hi, const uint64_t *keys, int32_t leaf_max,
                              int32_t *nch, int32_t *bnd, int32_t *nsplit) {
  const int32_t c = lo + static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= hi) return;
  const int32_t *C = cell + static_cast<size_t>(c) * kCellInts;
  const int32_t L = C[0], b = C[4], e = C[5];
  int32_t *B = bnd + static_cast<size_t>(c - lo) * 9;
  int32_t cnt = 0;
  if (e - b > leaf_max && L < kBits) {
    const int shift = 3 * (kBits - 1 - L);
    B[0] = b;
    for (int oct = 1; oct < 8; ++oct) {
      int32_t l = B[oct - 1], r = e;  // first position whose octant digit >= oct
      while (l < r) {
        const int32_t m = l + (r - l) / 2;
        if (static_cast<int>((keys[m] >> shift) & 7u) < oct) l = m + 1;
        else r = m;
      }
      B[oct] = l;
    }
    B[8] = e;
    for (int oct = 0; oct < 8; ++oct) cnt += (B[oct + 1] > B[oct]) ? 1 : 0;
    const uint64_t m = ballot(true);  // the lanes whose cells split
    if (static_cast<int>(lane_id()) == __builtin_ctzll(m)) atomicAdd(nsplit, __popcll(m));
  }
  nch[c - lo] = cnt;
}

// Exclusive scan of nch[0, m) in one workgroup of 1024 threads; *total gets the sum.
__global__ __launch_bounds__(1024) void k_scan(const int32_t *nch, int32_t *off, int32_t m, int32_t *total) {
  __shared__ int32_t part[1024];
  const int32_t t = threadIdx.x;
  const int32_t per = (m + 1023) / 1024;
  const int32_t b = t * per, e = min(m, b + per);
  int32_t s = 0;
  for (int32_t i = b; i < e; ++i) s += nch[i];
  part[t] = s;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const int32_t v = t >= d ? part[t - d] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int32_t run = part[t] - s;
  for (int32_t i = b; i < e; ++i) {
    off[i] = run;
    run += nch[i];
  }
  if (t == 1023) *total = part[1023];
}

__global__ void k_level_write(int32_t *cell, int32_t *parent, int32_t lo, int32_t hi, const int32_t *nch,
                              const int32_t *off, const int32_t *bnd) {
  const int32_t c = lo + static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= hi) return;
  int32_t *C = cell + static_cast<size_t>(c) * kCellInts;
  const int32_t k = nch[c - lo];
  const int32_t first = hi + off[c - lo];
  C[6] = k ? first : 0;
  C[7] = k;
  if (!k) return;
  const int32_t *B = bnd + static_cast<size_t>(c - lo) * 9;
  const int32_t L = C[0], half = 1 << (kBits - 1 - L);
  int32_t w = first;
  for (int oct = 0; oct < 8; ++oct) {
    if (B[oct + 1] == B[oct]) continue;
    int32_t *D = cell + static_cast<size_t>(w) * kCellInts;
    D[0] = L + 1;
    D[1] = C[1] + ((oct >> 2) & 1) * half;
    D[2] = C[2] + ((oct >> 1) & 1) * half;
    D[3] = C[3] + (oct & 1) * half;
    D[4] = B[oct];
    D[5] = B[oct + 1];
    D[6] = 0;
    D[7] = 0;
    parent[w] = c;
    ++w;
  }
}

// ---- translations -----------------------------------------------------------------
// Binomial re-centring of a cell's 84 coefficients held in registers, one axis
// after another (every index is a compile-time constant): 126 multiply-adds
// an axis instead of the full triple sum's 1,716 (M2M) per coefficient set.
constexpr Tables kHostTab = make_tables();

template <int AXIS>
GTAP_DEV void shift_moments(double *q, double s) {  // Q'_b = sum_i C(b, i) s^(b - i) Q_i
  double pw[kP + 1];
  pw[0] = 1.0;
#pragma unroll
  for (int i = 1; i <= kP; ++i) pw[i] = pw[i - 1] * s;
#pragma unroll
  for (int e = kP; e >= 1; --e) {  // descending: the lower exponents are still the old ones
#pragma unroll
    for (int t = 0; t < kNc; ++t) {
      if (kHostTab.e[t][AXIS] != e) continue;
      double acc = q[t];
      int u = t;
#pragma unroll
      for (int i = e - 1; i >= 0; --i) {
        u = kHostTab.dm1[u][AXIS];
        acc += (kHostTab.binom[e][i] * pw[e - i]) * q[u];
      }
      q[t] = acc;
    }
  }
}
template <int AXIS>
GTAP_DEV void shift_locals(double *l, double s) {  // L'_v = sum_i C(i, v) s^(i - v) L_i
  double pw[kP + 1];
  pw[0] = 1.0;
#pragma unroll
  for (int i = 1; i <= kP; ++i) pw[i] = pw[i - 1] * s;
#pragma unroll
  for (int e = 0; e < kP; ++e) {  // ascending: the higher exponents are still the old ones
#pragma unroll
    for (int t = 0; t < kNc; ++t) {
      if (kHostTab.e[t][AXIS] != e) continue;
      double acc = l[t];
#pragma unroll
      for (int i = e + 1; i <= kP; ++i) {
        const int d = kHostTab.deg[t] - e + i;
        if (d > kP) continue;
        const int u = kHostTab.idx[AXIS == 0 ? i : kHostTab.e[t][0]][AXIS == 1 ? i : kHostTab.e[t][1]]
                                  [AXIS == 2 ? i : kHostTab.e[t][2]];
        acc += (kHostTab.binom[i][e] * pw[i - e]) * l[u];
      }
      l[t] = acc;
    }
  }
}

// The 84 coefficients of one cell, 16 bytes at a time (rows are 672 bytes).
GTAP_DEV void load_coefs(const double *src, double *v) {
  const double2 *p = reinterpret_cast<const double2 *>(src);
#pragma unroll
  for (int t = 0; t < kNc / 2; ++t) {
    const double2 x = p[t];
    v[2 * t] = x.x;
    v[2 * t + 1] = x.y;
  }
}

// Reduced moments of every cell (see the top of the file), one cell per lane.
__global__ __launch_bounds__(64) void k_reduce_moments(const double *Q, double *Qr, int32_t ncells) {
  const int32_t c = static_cast<int32_t>(blockIdx.x * 64u + threadIdx.x);
  if (c >= ncells) return;
  double q[kNc];
  load_coefs(Q + static_cast<size_t>(c) * kNc, q);
#pragma unroll
  for (int t = 0; t < kNc; ++t) q[t] *= ((kHostTab.deg[t] & 1) ? -1.0 : 1.0) / kHostTab.fact[t];
#pragma unroll
  for (int z = kP; z >= 2; --z) {
#pragma unroll
    for (int t = 0; t < kNc; ++t) {
      if (kHostTab.e[t][2] != z) continue;
      q[kHostTab.idx[kHostTab.e[t][0] + 2][kHostTab.e[t][1]][z - 2]] -= q[t];
      q[kHostTab.idx[kHostTab.e[t][0]][kHostTab.e[t][1] + 2][z - 2]] -= q[t];
    }
  }
  double *dst = Qr + static_cast<size_t>(c) * kQrStride;
#pragma unroll
  for (int r = 0; r < kNr; ++r) dst[qr_at(r)] = q[kHostTab.red[r]];
}

// Add a cell's local coefficients to l from its reduced ones.
GTAP_DEV void add_reduced_locals(const double *src, double *l) {
  double v[kNc];
#pragma unroll
  for (int r = 0; r < kNr; ++r) v[kHostTab.red[r]] = src[r];
#pragma unroll
  for (int z = 2; z <= kP; ++z) {
#pragma unroll
    for (int t = 0; t < kNc; ++t) {
      if (kHostTab.e[t][2] != z) continue;
      v[t] = -(v[kHostTab.idx[kHostTab.e[t][0] + 2][kHostTab.e[t][1]][z - 2]] +
               v[kHostTab.idx[kHostTab.e[t][0]][kHostTab.e[t][1] + 2][z - 2]]);
    }
  }
#pragma unroll
  for (int t = 0; t < kNc; ++t) l[t] += v[t] * (1.0 / kHostTab.fact[t]);
}

// Sum over the 8 lanes of an aligned group, by DPP.
template <int CTRL>
GTAP_DEV double dpp_add(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint64_t y = dpp_in64<CTRL, 0xF>(b);
  return x + __builtin_bit_cast(double, y);
}
GTAP_DEV double sum8(double x) {
  x = dpp_add<0xB1>(x);   // lane ^ 1
  x = dpp_add<0x4E>(x);   // lane ^ 2
  return dpp_add<0x141>(x);  // lane ^ 7 (every quad already holds its sum)
}

// ---- upward pass ----------------------------------------------------------------
// P2M for the leaves among cells [lo, hi): one wavefront per cell.  The powers
// of 64 points' offsets go to LDS (one point per lane); lane t then sums the
// monomials t and t + 64 over the points.
__global__ __launch_bounds__(64) void k_p2m(const int32_t *cell, int32_t lo, int32_t hi, const double *px,
                                            const double *py, const double *pz, const double *pq, double *Q) {
  const int32_t c = lo + static_cast<int32_t>(blockIdx.x);
  if (c >= hi) return;
  const int32_t *C = cell + static_cast<size_t>(c) * kCellInts;
  if (C[7] != 0) return;
  __shared__ double pw[3][kP + 1][kWave];
  const double cx = cell_centre(C[1], C[0]), cy = cell_centre(C[2], C[0]), cz = cell_centre(C[3], C[0]);
  const int t = threadIdx.x, t2 = t + 64 < kNc ? t + 64 : t;
  const int e[2][3] = {{kTab.e[t][0], kTab.e[t][1], kTab.e[t][2]}, {kTab.e[t2][0], kTab.e[t2][1], kTab.e[t2][2]}};
  double acc0 = 0.0, acc1 = 0.0;
  for (int32_t b = C[4]; b < C[5]; b += static_cast<int32_t>(kWave)) {
    const int32_t k = b + t;
    if (k < C[5]) {
      const double d[3] = {px[k] - cx, py[k] - cy, pz[k] - cz};
      double x = pq[k], y = 1.0, z = 1.0;  // the charge travels with x
#pragma unroll
      for (int i = 0; i <= kP; ++i) {
        pw[0][i][t] = x;
        pw[1][i][t] = y;
        pw[2][i][t] = z;
        x *= d[0];
        y *= d[1];
        z *= d[2];
      }
    }
    __syncthreads();
    const int m = min(static_cast<int>(kWave), C[5] - b);
    for (int j = 0; j < m; ++j) {
      acc0 += pw[0][e[0][0]][j] * pw[1][e[0][1]][j] * pw[2][e[0][2]][j];
      acc1 += pw[0][e[1][0]][j] * pw[1][e[1][1]][j] * pw[2][e[1][2]][j];
    }
    __syncthreads();
  }
  Q[static_cast<size_t>(c) * kNc + t] = acc0;
  if (t + 64 < kNc) Q[static_cast<size_t>(c) * kNc + t + 64] = acc1;
}

// M2M for the internal cells among [lo, hi) (children already final): eight
// lanes per cell, a child on each, its moments re-centred in registers and
// summed over the lanes.
__global__ __launch_bounds__(256) void k_m2m(const int32_t *cell, int32_t lo, int32_t hi, double *Q) {
  const int32_t g = static_cast<int32_t>((blockIdx.x * 256u + threadIdx.x) / 8);
  const int32_t k = static_cast<int32_t>(threadIdx.x % 8);
  const int32_t c = lo + g;
  int32_t nch = 0, first = 0;
  const int32_t *C = cell + static_cast<size_t>(c < hi ? c : lo) * kCellInts;
  if (c < hi) {
    nch = C[7];
    first = C[6];
  }
  if (ballot(nch > 0) == 0ull) return;  // wave-uniform: the sums below need every lane
  double q[kNc];
#pragma unroll
  for (int t = 0; t < kNc; ++t) q[t] = 0.0;
  if (k < nch) {
    const int32_t ch = first + k;
    const int32_t *D = cell + static_cast<size_t>(ch) * kCellInts;
    load_coefs(Q + static_cast<size_t>(ch) * kNc, q);
    shift_moments<0>(q, cell_centre(D[1], D[0]) - cell_centre(C[1], C[0]));
    shift_moments<1>(q, cell_centre(D[2], D[0]) - cell_centre(C[2], C[0]));
    shift_moments<2>(q, cell_centre(D[3], D[0]) - cell_centre(C[3], C[0]));
  }
  double *dst = Q + static_cast<size_t>(c) * kNc;
#pragma unroll
  for (int t = 0; t < kNc; ++t) {
    const double v = sum8(q[t]);
    if (nch > 0 && k == (t & 7)) dst[t] = v;
  }
}

// ---- downward pass --------------------------------------------------------------
// Local coefficients of the cells [lo, hi): M2L's sums (reduced) and, below the
// root, L2L from the parents (already final), one cell per lane, re-centred
// in registers.
__global__ __launch_bounds__(64) void k_l2l(const int32_t *cell, const int32_t *parent, int32_t lo, int32_t hi,
                                            const double *Lr, double *L) {
  const int32_t c = lo + static_cast<int32_t>(blockIdx.x * 64u + threadIdx.x);
  if (c >= hi) return;
  const int32_t pc = parent[c];
  double l[kNc];
#pragma unroll
  for (int t = 0; t < kNc; ++t) l[t] = 0.0;
  if (pc >= 0) {
    const int32_t *C = cell + static_cast<size_t>(c) * kCellInts;
    const int32_t *P = cell + static_cast<size_t>(pc) * kCellInts;
    load_coefs(L + static_cast<size_t>(pc) * kNc, l);
    shift_locals<0>(l, cell_centre(C[1], C[0]) - cell_centre(P[1], P[0]));
    shift_locals<1>(l, cell_centre(C[2], C[0]) - cell_centre(P[2], P[0]));
    shift_locals<2>(l, cell_centre(C[3], C[0]) - cell_centre(P[3], P[0]));
  }
  add_reduced_locals(Lr + static_cast<size_t>(c) * kNr, l);
  double2 *dst = reinterpret_cast<double2 *>(L + static_cast<size_t>(c) * kNc);
#pragma unroll
  for (int t = 0; t < kNc / 2; ++t) dst[t] = make_double2(l[2 * t], l[2 * t + 1]);
}

// L2P for the leaves among [lo, hi): one wavefront per leaf, a point per lane;
// the leaf's coefficients are wave-uniform, nested in x, y, z.
__global__ __launch_bounds__(64) void k_l2p(const int32_t *cell, int32_t lo, int32_t hi, const double *L,
                                            const double *px, const double *py, const double *pz, double *phi) {
  const int32_t c = lo + static_cast<int32_t>(blockIdx.x);
  if (c >= hi) return;
  const int32_t *C = cell + static_cast<size_t>(c) * kCellInts;
  if (C[7] != 0) return;
  const double *l = L + static_cast<size_t>(c) * kNc;
  const double cx = cell_centre(C[1], C[0]), cy = cell_centre(C[2], C[0]), cz = cell_centre(C[3], C[0]);
  for (int32_t k = C[4] + static_cast<int32_t>(threadIdx.x); k < C[5]; k += static_cast<int32_t>(kWave)) {
    const double dx = px[k] - cx, dy = py[k] - cy, dz = pz[k] - cz;
    double sx = 0.0;
#pragma unroll
    for (int i = kP; i >= 0; --i) {
      double sy = 0.0;
#pragma unroll
      for (int j = kP - i; j >= 0; --j) {
        double sz = 0.0;
#pragma unroll
        for (int m = kP - i - j; m >= 0; --m) sz = sz * dz + l[kHostTab.idx[i][j][m]];
        sy = sy * dy + sz;
      }
      sx = sx * dx + sy;
    }
    phi[k] += sx;
  }
}

__global__ void k_scatter(int32_t n, const int32_t *perm, const double *phi_sorted, double *phi) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) phi[perm[k]] = phi_sorted[k];
}

}  // namespace fmm
}  // namespace gtap
