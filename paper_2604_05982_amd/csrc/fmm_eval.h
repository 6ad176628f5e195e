// fmm_eval.h -- evaluation of the sorted FMM interaction lists (GTaP Sec.
// 6.4.1 names the phases): M2L into the local expansions, P2P into the
// potentials.  The lists come from the traversals of fmm_lists.h, sorted by
// target cell.
//
// MI355X choices: M2L gives each target one wavefront, one source per lane,
// and adds its sums once.  P2P is balanced over the list entries instead (64
// per wavefront), because a target leaf's segment can be tens of thousands of
// entries long; the wavefronts that share a target add their potentials with
// fp64 atomics.
#pragma once
#include "fmm_lists.h"

namespace gtap {
namespace fmm {

constexpr uint32_t kM2LThreads = 64;

// Workgroup -> M2L target.  Workgroups go round-robin to the eight XCDs, each
// with an L2 of its own; runs of kM2LRun consecutive targets stay on one XCD, so
// that neighbours find the sources they share there.  The grid is a multiple of
// 8 * kM2LRun (positions past the end have no work).  Runs must be short next to
// the tree, or small jobs leave XCDs idle: k_m2l_list with runs of 1, 16, 64 and
// 256 takes 23, 23, 23 and 31 us for 504 cells (10,000 points), 156, 157, 160
// and 159 us for 6,260, and 3.86, 3.82, 3.78 and 3.77 ms for 145,571 (4 M
// points).  P2P gains nothing from runs (16.8 ms for 4 M points with and
// without; runs of 64 workgroups: 0.11 -> 0.16 ms for 10,000).
constexpr uint32_t kXcds = 8;
constexpr uint32_t kM2LRun = 16;
GTAP_DEV uint32_t m2l_target(uint32_t block) {
  const uint32_t xcd = block % kXcds, i = block / kXcds;
  return (i / kM2LRun * kXcds + xcd) * kM2LRun + i % kM2LRun;
}

// The 49 derivatives T'_g = d^g (1/|d|) with g_z <= 1 (|g| <= 6), times `unit`:
// the Coulomb three-term recurrence multiplied by g! becomes
// T'_g = -[(2n-1) sum_i g_i d_i T'_{g-e_i} + (n-1) sum_i g_i (g_i - 1) T'_{g-2e_i}] / (n r^2),
// n = |g|, closed on g_z <= 1.  Fully unrolled, T' stays in registers.
GTAP_DEV void taylor_scaled(double d0, double d1, double d2, double unit, double *T) {
  const double inv_r2 = 1.0 / (d0 * d0 + d1 * d1 + d2 * d2);
  T[0] = unit * sqrt(inv_r2);
  const double dd[3] = {d0, d1, d2};
#pragma unroll
  for (int g = 1; g < kNr; ++g) {
    const int x = kHostTab.ge[g][0], y = kHostTab.ge[g][1], z = kHostTab.ge[g][2];
    const double n = static_cast<double>(x + y + z);
    double s1 = 0.0, s2 = 0.0;
    if (x >= 1) s1 += x * dd[0] * T[kHostTab.g_of[x >= 1 ? x - 1 : 0][y][z]];
    if (y >= 1) s1 += y * dd[1] * T[kHostTab.g_of[x][y >= 1 ? y - 1 : 0][z]];
    if (z >= 1) s1 += z * dd[2] * T[kHostTab.g_of[x][y][z >= 1 ? z - 1 : 0]];
    if (x >= 2) s2 += x * (x - 1) * T[kHostTab.g_of[x >= 2 ? x - 2 : 0][y][z]];
    if (y >= 2) s2 += y * (y - 1) * T[kHostTab.g_of[x][y >= 2 ? y - 2 : 0][z]];
    T[g] = -((2.0 * n - 1.0) / n * s1 + (n - 1.0) / n * s2) * inv_r2;
  }
}

// Lane sums of 64 values (v[i] on every lane; those from kNr on are zero):
// lane i returns the sum of v[i] over the lanes.  Each round adds the lanes at
// distance 32, 16, ..., 1 and keeps half of the values.
template <int D>
GTAP_DEV double pair_sum(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  if constexpr (D >= 16) {
    // the swap leaves a of the lower and b of the upper lanes of each pair in
    // the first result, their partners in the second
    uint32_t r0[2], r1[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t xh = static_cast<uint32_t>(x >> (32 * h)), yh = static_cast<uint32_t>(y >> (32 * h));
      const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false)
                             : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
      r0[h] = r[0];
      r1[h] = r[1];
    }
    return __builtin_bit_cast(double, (static_cast<uint64_t>(r0[1]) << 32) | r0[0]) +
           __builtin_bit_cast(double, (static_cast<uint64_t>(r1[1]) << 32) | r1[0]);
  } else {
    double sa, sb;
    if constexpr (D == 8) {
      sa = dpp_add<0x128>(a);  // row_ror:8
      sb = dpp_add<0x128>(b);
    } else if constexpr (D == 4) {  // half-row mirror of the quads reversed: lane ^ 4
      sa = a + __builtin_bit_cast(double, dpp_in64<0x1B, 0xF>(dpp_in64<0x141, 0xF>(x)));
      sb = b + __builtin_bit_cast(double, dpp_in64<0x1B, 0xF>(dpp_in64<0x141, 0xF>(y)));
    } else if constexpr (D == 2) {
      sa = dpp_add<0x4E>(a);
      sb = dpp_add<0x4E>(b);
    } else {
      sa = dpp_add<0xB1>(a);
      sb = dpp_add<0xB1>(b);
    }
    return (lane_id() & D) ? sb : sa;
  }
}
template <int D, int N>
GTAP_DEV double scatter_sums(double *v) {  // N = 2 D values
#pragma unroll
  for (int i = 0; i < D; ++i) v[i] = pair_sum<D>(v[i], v[i + D]);
  if constexpr (D > 1) return scatter_sums<D / 2, D>(v);
  else return v[0];
}

// The terms of one half (moments of degree <= 4, then 5 and 6) of a lane's row.
template <int HALF>
GTAP_DEV void m2l_terms(const double2 *row, const double (&T)[kNr], double (&acc)[kWave]) {
  constexpr int b0 = HALF ? nred(4) : 0, nb = HALF ? kNr - nred(4) : nred(4);
#pragma unroll
  for (int i = 0; i < nb; ++i) {
    const int tb = kHostTab.red[b0 + i];
    const double2 pair = row[i / 2];
    const double qb = (i & 1) ? pair.y : pair.x;
#pragma unroll
    for (int ra = 0; ra < nred(kP - kHostTab.deg[tb]); ++ra) {
      const int ta = kHostTab.red[ra];
      const int x = kHostTab.e[ta][0] + kHostTab.e[tb][0], y = kHostTab.e[ta][1] + kHostTab.e[tb][1],
                z = kHostTab.e[ta][2] + kHostTab.e[tb][2];
      if (z < 2) {
        acc[ra] += T[kHostTab.g_of[x][y][z < 2 ? z : 0]] * qb;
      } else {
        acc[ra] -= T[kHostTab.g_of[z < 2 ? x : x + 2][y][0]] * qb;
        acc[ra] -= T[kHostTab.g_of[x][z < 2 ? y : y + 2][0]] * qb;
      }
    }
  }
}

// M2L over the sorted list: one wavefront per target cell, 64 sources at a
// time, one per lane.  A lane keeps its source's 49 derivatives and its 49 sums
// in registers and adds T'_{a+b} Q'_b for every term (the 70 with g_z = 2 as
// minus the sum of two): 602 fused multiply-adds, all indices compile-time
// constants.  The sources' reduced moments come through LDS, half a row (26
// doubles, 13 x 16 bytes) at a time by direct loads that need no registers, so
// that all 13 are in flight and eight wavefronts fit a compute unit.  67 M pairs
// of 4 M uniform points: 13.6 ms with the full sets (84 + 84 coefficients, rows
// read by their own lanes, 64 lines per load, half the registers reached by
// moves), 11.0 ms with reduced sets and runs of targets per XCD, 3.8 ms with
// direct loads; what is left is the fp64 VALU and the wait for the two halves.
__global__ __launch_bounds__(kM2LThreads, 2) void k_m2l_list(const int32_t *__restrict__ cell,
                                                             const double *__restrict__ Qr, double *Lr,
                                                             const uint64_t *__restrict__ pairs,
                                                             const uint64_t *__restrict__ seg_lo,
                                                             const uint64_t *__restrict__ seg_hi, uint32_t ncells) {
  constexpr int kHalf = kQrStride / 2;            // doubles of half a row: degrees <= 4, then 5 and 6
  constexpr uint32_t kUnits = kHalf / 2;          // 16-byte units of it
  static_assert(kHalf % 2 == 0 && kHalf >= nred(4) && kHalf >= kNr - nred(4), "halves of a row");
  __shared__ double2 rows[kWave * kUnits];
  const uint32_t a = m2l_target(blockIdx.x);
  if (a >= ncells) return;
  const uint64_t lo = seg_lo[a], hi = seg_hi[a];
  const uint32_t ln = threadIdx.x;
  if (lo == hi) {
    if (ln < static_cast<uint32_t>(kNr)) Lr[static_cast<size_t>(a) * kNr + ln] = 0.0;
    return;
  }
  int32_t A[kCellInts];
  load_cell(cell, a, A);
  const double cx = cell_centre(A[1], A[0]), cy = cell_centre(A[2], A[0]), cz = cell_centre(A[3], A[0]);
  double acc[kWave];
#pragma unroll
  for (int t = 0; t < static_cast<int>(kWave); ++t) acc[t] = 0.0;
  for (uint64_t s0 = lo; s0 < hi; s0 += kWave) {
    const uint32_t n = static_cast<uint32_t>(min(static_cast<uint64_t>(kWave), hi - s0));
    // lanes past the end repeat the first source with zero derivatives
    const uint32_t b = static_cast<uint32_t>(pairs[s0 + (ln < n ? ln : 0u)]);
    auto stage = [&](int half) {
      // The loads write LDS when they return, in no order with the LDS reads
      // before them: every earlier read of `rows` completes first.
      drain();
      uint32_t l = ln;
      asm volatile("" : "+v"(l));  // the 13 addresses are formed here, not kept in registers across the loop
#pragma unroll
      for (uint32_t j = 0; j < kUnits; ++j) {
        const uint32_t unit = j * kWave + l, row = unit / kUnits;
        const uint32_t src = static_cast<uint32_t>(__shfl(static_cast<int>(b), static_cast<int>(row), 64));
        const double *g = Qr + static_cast<size_t>(src) * kQrStride + half * kHalf + 2 * (unit - row * kUnits);
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const __attribute__((address_space(1))) uint32_t *>(
                                             reinterpret_cast<uintptr_t>(g)),
                                         reinterpret_cast<__attribute__((address_space(3))) uint32_t *>(
                                             static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&rows[j * kWave]))),
                                         16, 0, 0);
      }
    };
    stage(0);
    int32_t B[kCellInts];
    load_cell(cell, b, B);
    double T[kNr];
    taylor_scaled(cx - cell_centre(B[1], B[0]), cy - cell_centre(B[2], B[0]), cz - cell_centre(B[3], B[0]),
                  ln < n ? 1.0 : 0.0, T);
    drain();  // the rows are in LDS
    m2l_terms<0>(rows + ln * kUnits, T, acc);
    stage(1);
    drain();
    m2l_terms<1>(rows + ln * kUnits, T, acc);
  }
  const double v = scatter_sums<32, 64>(acc);
  if (ln < static_cast<uint32_t>(kNr)) Lr[static_cast<size_t>(a) * kNr + ln] = v;
}

constexpr uint32_t kP2PThreads = 256;
constexpr uint32_t kP2PTileL = 64;
constexpr double kOutside = 1024.0;  // an x coordinate outside the root cube

// P2P over the sorted list, balanced over its entries: wavefront w takes the
// 64 entries 64 w .. 64 w + 63 (one per lane), so a target whose segment is
// long (a large leaf next to a dense region meets tens of thousands of source
// leaves) is spread over many wavefronts, and adds its potentials atomically.
// The entries form runs of one target.  Per run, the sources of its leaves
// are concatenated (exclusive prefix of the leaf sizes over the run's lanes)
// and walked in chunks of 64 points: the owner of chunk position c is the
// last leaf starting at or before it (marks in LDS and a prefix maximum), each
// lane loads one point, the chunk is staged in LDS as (x, y, z, q), and the
// next chunk is loaded while this one is evaluated.  A tile of at most 64
// targets is padded to 2 P, P a power of two; the lanes form 64 / P groups of P,
// a lane holds the targets (lane mod P) and that + P, group g takes the chunk's
// sources g, g + 64/P, ..., and the groups' partial sums meet by lane shuffles.
// Two targets per source read, one refinement step of third order (rsqrt_h)
// and no tests in the loop: what bounds it is the fp64 VALU, 21.3 G
// interactions of 4 M uniform points took 25.6 ms with one target, two
// Newton-Raphson steps and the tests, 16.7 ms this way.  Distance zero needs a test only where
// the source chunk holds points of the target's own leaf: points at one place
// share a Morton key, so they share the leaf.  Chunks are padded with charge 0
// at a place outside the cube.  Interactions are counted, and coincident pairs
// as the pairs at distance zero less the points' meetings with themselves (one
// per target point and self pair).
__global__ __launch_bounds__(kP2PThreads) void k_p2p_list(const int32_t *__restrict__ cell,
                                                          const double *__restrict__ px,
                                                          const double *__restrict__ py,
                                                          const double *__restrict__ pz,
                                                          const double *__restrict__ pq, double *phi,
                                                          const uint64_t *__restrict__ pairs, uint64_t n,
                                                          uint32_t ncells, uint64_t *inter_out, uint64_t *coinc_out) {
  constexpr uint32_t W = kP2PThreads / kWave;
  __shared__ double2 stage[W][2 * kWave];
  __shared__ uint32_t mark[W][kWave];
  const uint32_t tx = threadIdx.x, ln = tx % kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(tx / kWave);
  const uint64_t e0 = (static_cast<uint64_t>(blockIdx.x) * W + wv) * kWave;
  if (e0 >= n) return;
  const uint32_t ne = static_cast<uint32_t>(min(static_cast<uint64_t>(kWave), n - e0));
  double2 *const st = stage[wv];
  uint32_t *const mk = mark[wv];
  // entry e0 + ln: target ta (ncells for the gaps, which sort last, and past
  // the end), source leaf sb with points rb .. rb + rn - 1, target points
  // tb .. tb + tn - 1
  uint32_t ta = ncells, sb = 0;
  int32_t rb = 0, rn = 0, tb = 0, tn = 0;
  if (ln < ne) {
    const uint64_t e = pairs[e0 + ln];
    if (static_cast<uint32_t>(e >> 32) < ncells) {
      ta = static_cast<uint32_t>(e >> 32);
      sb = static_cast<uint32_t>(e);
      rb = cell[static_cast<size_t>(sb) * kCellInts + 4];
      rn = cell[static_cast<size_t>(sb) * kCellInts + 5] - rb;
      tb = cell[static_cast<size_t>(ta) * kCellInts + 4];
      tn = cell[static_cast<size_t>(ta) * kCellInts + 5] - tb;
    }
  }
  const uint32_t nv = static_cast<uint32_t>(__popcll(ballot(ta < ncells)));
  uint64_t inter = 0, selfm = 0;
  uint32_t zc = 0;
  for (uint32_t k0 = 0; k0 < nv;) {
    // the run of target a: lanes k0 .. k1 - 1
    const uint32_t a = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(ta), static_cast<int>(k0)));
    const uint64_t other = ballot(ta != a) & (~0ull << k0);
    const uint32_t k1 = other ? static_cast<uint32_t>(__builtin_ctzll(other)) : kWave;
    const bool in_run = ln >= k0 && ln < k1;
    const int32_t rn_run = in_run ? rn : 0;
    const int32_t incl = static_cast<int32_t>(wave_inclusive_sum(static_cast<uint32_t>(rn_run)));
    const int32_t pre = incl - rn_run;  // first concatenated position of this lane's leaf
    const int32_t stotal = __builtin_amdgcn_readlane(incl, static_cast<int>(k1 - 1));
    const int32_t ab = __builtin_amdgcn_readlane(tb, static_cast<int>(k0));
    const int32_t na = __builtin_amdgcn_readlane(tn, static_cast<int>(k0));
    const uint32_t nself = static_cast<uint32_t>(__popcll(ballot(in_run && sb == a)));
    inter += static_cast<uint64_t>(static_cast<int64_t>(na) * stotal - static_cast<int64_t>(nself) * na);
    selfm += static_cast<uint64_t>(nself) * static_cast<uint64_t>(na);
    // Loads chunk c's points into (sx, sy, sz, sq).
    double sx = 0.0, sy = 0.0, sz = 0.0, sq = 0.0;
    auto fetch = [&](int32_t c) {
      mk[ln] = 0;
      wave_sync();
      if (in_run && rn > 0 && pre < c + static_cast<int32_t>(kWave) && pre + rn > c)
        mk[pre > c ? pre - c : 0] = ln + 1;
      wave_sync();
      const uint32_t m = wave_inclusive_max(mk[ln]);
      wave_sync();
      const int32_t own = m ? static_cast<int32_t>(m) - 1 : 0;
      const int32_t ob = __shfl(rb, own, 64), op = __shfl(pre, own, 64);
      const int32_t pos = c + static_cast<int32_t>(ln);
      // past the end: no charge, and outside the cube [-128, 128)^3
      sx = kOutside;
      sy = sz = sq = 0.0;
      if (pos < stotal) {
        const int32_t sj = ob + (pos - op);
        sx = px[sj];
        sy = py[sj];
        sz = pz[sj];
        sq = pq[sj];
      }
    };
    // positions of the target's own leaf among the sources (every self entry)
    const bool is_self = in_run && sb == a;
    for (int32_t t0 = 0; t0 < na; t0 += static_cast<int32_t>(kP2PTileL)) {
      const int32_t nt = min(static_cast<int32_t>(kP2PTileL), na - t0);
      uint32_t P = 1;
      while (2 * P < static_cast<uint32_t>(nt)) P <<= 1;
      const int32_t ng = static_cast<int32_t>(kWave / P);
      const uint32_t tl = ln & (P - 1);
      const int32_t grp = static_cast<int32_t>(ln / P);
      const int32_t i0 = ab + t0 + static_cast<int32_t>(tl), i1 = i0 + static_cast<int32_t>(P);
      const bool live0 = static_cast<int32_t>(tl) < nt, live1 = static_cast<int32_t>(tl + P) < nt;
      // a lane without a target stands where no source is
      double x0 = live0 ? px[i0] : 2.0 * kOutside, y0 = live0 ? py[i0] : 0.0, z0 = live0 ? pz[i0] : 0.0;
      double x1 = live1 ? px[i1] : 2.0 * kOutside, y1 = live1 ? py[i1] : 0.0, z1 = live1 ? pz[i1] : 0.0;
      // taken as written here, so that the source loop's waits do not cover
      // the source prefetch
      asm volatile("" : "+v"(x0), "+v"(y0), "+v"(z0), "+v"(x1), "+v"(y1), "+v"(z1));
      double acc0 = 0.0, acc1 = 0.0;
      fetch(0);
      for (int32_t c0 = 0; c0 < stotal; c0 += static_cast<int32_t>(kWave)) {
        const int32_t cnt = min(static_cast<int32_t>(kWave), stotal - c0);
        st[2 * ln] = make_double2(sx, sy);
        st[2 * ln + 1] = make_double2(sz, sq);
        wave_sync();
        if (c0 + static_cast<int32_t>(kWave) < stotal) fetch(c0 + static_cast<int32_t>(kWave));
        const bool self_chunk = ballot(is_self && pre < c0 + static_cast<int32_t>(kWave) && pre + rn > c0) != 0ull;
        if (!self_chunk) {
          // u + grp < 64: u is a multiple of ng below cnt <= 64, grp < ng
#pragma unroll 4
          for (int32_t u = 0; u < cnt; u += ng) {
            const double2 s01 = st[2 * (u + grp)], s23 = st[2 * (u + grp) + 1];
            const double dx0 = x0 - s01.x, dy0 = y0 - s01.y, dz0 = z0 - s23.x;
            const double dx1 = x1 - s01.x, dy1 = y1 - s01.y, dz1 = z1 - s23.x;
            acc0 += s23.y * rsqrt_h(dx0 * dx0 + dy0 * dy0 + dz0 * dz0);
            acc1 += s23.y * rsqrt_h(dx1 * dx1 + dy1 * dy1 + dz1 * dz1);
          }
        } else {
          for (int32_t u = 0; u < cnt; u += ng) {
            const double2 s01 = st[2 * (u + grp)], s23 = st[2 * (u + grp) + 1];
            const double dx0 = x0 - s01.x, dy0 = y0 - s01.y, dz0 = z0 - s23.x;
            const double dx1 = x1 - s01.x, dy1 = y1 - s01.y, dz1 = z1 - s23.x;
            const double r0 = dx0 * dx0 + dy0 * dy0 + dz0 * dz0, r1 = dx1 * dx1 + dy1 * dy1 + dz1 * dz1;
            acc0 += r0 == 0.0 ? 0.0 : s23.y * rsqrt_h(r0 == 0.0 ? 1.0 : r0);
            acc1 += r1 == 0.0 ? 0.0 : s23.y * rsqrt_h(r1 == 0.0 ? 1.0 : r1);
            zc += (r0 == 0.0 ? 1u : 0u) + (r1 == 0.0 ? 1u : 0u);
          }
        }
        wave_sync();  // the chunk's reads are issued before the next one overwrites it
      }
      for (uint32_t d = P; d < kWave; d <<= 1) {
        acc0 += __shfl_xor(acc0, static_cast<int>(d), 64);
        acc1 += __shfl_xor(acc1, static_cast<int>(d), 64);
      }
      if (grp == 0) {
        if (live0) unsafeAtomicAdd(phi + i0, acc0);
        if (live1) unsafeAtomicAdd(phi + i1, acc1);
      }
    }
    k0 = k1;
  }
  const uint64_t coinc = readlane64(wave_inclusive_sum64(zc), 63) - selfm;
  if (ln == 0 && inter) fetch_add_relaxed(inter_out, inter);
  if (ln == 0 && coinc) fetch_add_relaxed(coinc_out, coinc);
}

}  // namespace fmm
}  // namespace gtap
