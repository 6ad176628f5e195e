// kclique_wave.h -- the split k-clique bodies (TK_KS_*), executed by the whole
// wavefront; the search itself is described in kclique_bits.h.
//
// A lane whose task is a row, a vertex counted in place, an edge, a heavy
// edge's root or a branch only describes it; the wavefront then runs the
// described tasks together, work spread over the lanes by a prefix sum.  Run
// by one lane each, 64 tasks took as long as the slowest: list searches were
// chains of dependent loads per lane and the private 64 x 64 matrices and
// stacks lived in scratch memory (1 M vertices, mean degree 40, k = 7,
// orientation: 64 rows 582 k cycles, 64 edges 801 k, 64 branches 509 k, 64
// vertices in place 2.2 M; VALU lane utilisation 23 %): 88 ms per call, this way
// 36 ms (rows 247 k, edges and branches 160 k, vertices in place 1.0 M; all
// now bound by load and LDS latency with one wavefront per SIMD), 28 ms with
// the scheduler of today.  100,003 vertices, mean degree 30, k = 6, pivoting:
// 17-21 -> 6.6 -> 5.3 ms.
//
//   rows (and the rows of vertices in place): either the members of N+(u) are
//     searched in N+(x), x the i-th of them, or N+(x) in N+(u), whichever has
//     fewer needles.  Where N+(x) begins after x (as it does for every
//     x where ids ascend along the edges) only members after x can be in it.
//     The needles of 64 rows are one concatenated stream, 256 at a time, so
//     that four loads a lane are in flight and a lane's share does not depend
//     on its own row's length;
//   edges and branches: the vertex's matrix is staged in LDS once for its
//     tasks on the lanes (up to 384 out-neighbours; larger ones are read in
//     place).  Orientation, cliques of up to five members in an
//     edge's candidates (k <= 7): run_sets.  Otherwise one task at a time: its
//     candidates' rows are renumbered by ballots, one column per ballot, into
//     a 64 x 64 matrix in LDS (the columns are the reversed DAG's rows, which
//     has the same cliques), and the pairs (a, b in a's row), or pivoting the
//     root's branches, are dealt to the lanes.
#pragma once
#include "kclique_bits.h"
#include "layout.h"
#include "tasks.h"
#include "wave.h"

namespace gtap {

// Candidate tasks of the plain k-clique search (kEmitCand): C /\ N+(u) of every
// lane in `todo`, counted for the last level, else also written, in order, to
// the lane's frame for its children.  The lanes' candidates are one
// concatenated stream, 256 at a time: one device-coherent load each (they may
// be another wavefront's writes), then a bisection of N+(u), which is read-only
// input and served by the caches, with four searches a lane in flight.  Bound
// by load latency with one wavefront per SIMD.  A galloping walk by each lane
// went at the pace of the longest lists, with coherent reads among its
// dependent loads: 28 k cycles an iteration (k = 7 on 300,000 vertices),
// 19 k this way.
//
// A lane whose N+(u) is shorter than C streams N+(u) and bisects C: its
// searches are then chains of coherent loads, but streaming all of C for every
// short list takes the product of the two.  Kernel times, C always streamed ->
// the shorter list: a vertex with 4,000 out-neighbours of out-degree 1, k = 3,
// 5.57 -> 0.38 ms; 20,000 vertices of mean degree 30 in random order, k = 5,
// 2.74 -> 1.62 ms.  Turning only at half or a quarter of C's length measured the
// same or up to 8 % slower.
//
// From two rounds of the stream on, both lists are first cut to the elements
// between the other's ends (four bisections side by side, about one round's
// time): lists of neighbouring ids overlap in a part only, and there a walk that
// finds each element next to the one before needs few loads.  3,000 vertices
// joined to the next 128, k = 3: 1.09 ms walked, 1.67 without the cut, 1.14; k = 7
// on 300,000 vertices 59.1 -> 54.1 ms.  From four or eight rounds on: 55.4, 56.8.
GTAP_DEV void run_cands(const Params &p, uint32_t *mark, uint64_t todo, uint32_t tid, Outcome &o) {
  constexpr uint32_t kFlight = 4;  // 64-element chunks in flight
  constexpr uint32_t kCut = 2 * kFlight * kWave;  // elements streamed from which the lists are cut first
  const uint32_t ln = lane_id();
  const bool mine = ((todo >> ln) & 1u) != 0;
  const bool turn = mine && o.d[5] < o.d[4];
  // streamed: n elements at (d0, d1); searched: nb elements at (d2, d3)
  uint32_t n = mine && o.d[4] > 0 && o.d[5] > 0 ? (turn ? o.d[5] : o.d[4]) : 0u;
  uint32_t nb = mine ? (turn ? o.d[4] : o.d[5]) : 0u;
  uint32_t d0 = turn ? o.d[2] : o.d[0], d1 = turn ? o.d[3] : o.d[1];
  uint32_t d2 = turn ? o.d[0] : o.d[2], d3 = turn ? o.d[1] : o.d[3];
  const uint64_t turned = ballot(turn);
  const uint32_t left = o.nchild;  // levels left; 1: count only
  uint64_t dst = 0;
  if (n > 0 && left > 1) dst = reinterpret_cast<uint64_t>(frame_ptr(p, tid) + FW_BUF);
  uint32_t total = 0;
  uint32_t off = wave_exclusive_scan(n, &total);
  auto wave_max = [](uint32_t x) {
    for (uint32_t i = 1; i < kWave; i <<= 1) {
      const uint32_t y = static_cast<uint32_t>(__shfl_xor(static_cast<int>(x), static_cast<int>(i), 64));
      x = y > x ? y : x;
    }
    return uniform(x);
  };
  uint32_t longest = wave_max(nb);
  auto from = [](uint32_t x, uint32_t k) {
    return static_cast<uint32_t>(__shfl(static_cast<int>(x), static_cast<int>(k), 64));
  };
  auto read = [](bool coherent, const int32_t *a) { return coherent ? co_ld32i(a) : *a; };
  if (total >= kCut) {
    // at[0, 1]: the streamed list's elements from the other's first one on and
    // up to its last one; at[2, 3]: the other way round
    const int32_t *S = reinterpret_cast<const int32_t *>(pack(d0, d1));
    const int32_t *B = reinterpret_cast<const int32_t *>(pack(d2, d3));
    uint32_t at[4] = {0, 0, 0, 0};
    int32_t v[4] = {0, 0, 0, 0};
    if (n > 0) {
      v[0] = read(turn, B);
      v[1] = read(turn, B + nb - 1) + 1;
      v[2] = read(!turn, S);
      v[3] = read(!turn, S + n - 1) + 1;
    }
    const uint32_t top = wave_max(n > 0 ? (n > nb ? n : nb) : 1u);
    for (uint32_t step = 1u << (31 - __builtin_clz(top)); step > 0; step >>= 1) {
      int32_t y[4];
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t len = n > 0 ? (q < 2 ? n : nb) : 0u;
        y[q] = at[q] + step <= len ? read(q < 2 ? !turn : turn, (q < 2 ? S : B) + (at[q] + step - 1)) : 0x7FFFFFFF;
      }
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t len = n > 0 ? (q < 2 ? n : nb) : 0u;
        at[q] += at[q] + step <= len && y[q] < v[q] ? step : 0u;
      }
    }
    S += at[0];
    B += at[2];
    n = at[1] > at[0] && at[3] > at[2] ? at[1] - at[0] : 0u;
    nb = n > 0 ? at[3] - at[2] : 0u;
    const uint64_t s64 = reinterpret_cast<uint64_t>(S), b64 = reinterpret_cast<uint64_t>(B);
    d0 = static_cast<uint32_t>(s64); d1 = static_cast<uint32_t>(s64 >> 32);
    d2 = static_cast<uint32_t>(b64); d3 = static_cast<uint32_t>(b64 >> 32);
    off = wave_exclusive_scan(n, &total);
    longest = wave_max(nb);
  }
  uint32_t carry = 0, found = 0;
  for (uint32_t c0 = 0; c0 < total; c0 += kFlight * kWave) {
    uint32_t own[kFlight], at[kFlight], len[kFlight];
    int32_t x[kFlight];
    const int32_t *list[kFlight];
    bool co[kFlight];  // the searched list is C
#pragma unroll
    for (uint32_t q = 0; q < kFlight; ++q) {
      const uint32_t g0 = c0 + q * kWave;
      own[q] = chunk_owner(mark, n, off, g0, carry);
      const int32_t *src = reinterpret_cast<const int32_t *>(pack(from(d0, own[q]), from(d1, own[q])));
      list[q] = reinterpret_cast<const int32_t *>(pack(from(d2, own[q]), from(d3, own[q])));
      const uint32_t first = from(off, own[q]), nu = from(nb, own[q]);
      const bool act = g0 + ln < total;
      len[q] = act ? nu : 0u;
      at[q] = 0;
      co[q] = ((turned >> own[q]) & 1u) != 0;
      x[q] = act ? read(!co[q], src + (g0 + ln - first)) : 0;
    }
    // at[q]: elements of the list below x[q]
    for (uint32_t step = 1u << (31 - __builtin_clz(longest)); step > 0; step >>= 1) {
      int32_t y[kFlight];
#pragma unroll
      for (uint32_t q = 0; q < kFlight; ++q)
        y[q] = at[q] + step <= len[q] ? read(co[q], list[q] + (at[q] + step - 1)) : 0x7FFFFFFF;
#pragma unroll
      for (uint32_t q = 0; q < kFlight; ++q) at[q] += at[q] + step <= len[q] && y[q] < x[q] ? step : 0u;
    }
    bool hit[kFlight];
#pragma unroll
    for (uint32_t q = 0; q < kFlight; ++q) {
      const int32_t y = at[q] < len[q] ? read(co[q], list[q] + at[q]) : 0;
      hit[q] = at[q] < len[q] && y == x[q];
    }
#pragma unroll
    for (uint32_t q = 0; q < kFlight; ++q) {
      const uint32_t g0 = c0 + q * kWave;
      const uint64_t m = ballot(hit[q]);
      if (m == 0ull) continue;
      const uint64_t buf = pack(from(static_cast<uint32_t>(dst), own[q]), from(static_cast<uint32_t>(dst >> 32), own[q]));
      const uint32_t first = from(off, own[q]), before = from(found, own[q]);
      const uint32_t s0 = first > g0 ? first - g0 : 0u;  // the run's first position in the chunk
      if (hit[q] && buf != 0)
        co_st32i(reinterpret_cast<int32_t *>(buf) + before + rank_below(m & ~((1ull << s0) - 1)), x[q]);
      // this lane's run in the chunk: positions [a, b)
      const uint32_t a = off > g0 ? off - g0 : 0u, b = off + n > g0 ? off + n - g0 : 0u;
      if (a < b && a < kWave) {
        const uint64_t run = (b >= kWave ? ~0ull : (1ull << b) - 1) & ~((1ull << a) - 1);
        found += __popcll(m & run);
      }
    }
  }
  if (!mine) return;
  if (left == 1) {
    o.value = found;
    return;
  }
  o.words += found;  // the candidates written for the children
  if (found == 0) return;
  o.type = OUT_FORK;
  o.nchild = found;
  o.ckind = TK_KC_CAND;
  o.big = (left - 1 >= 2) ? 1u : 0u;
  o.d[0] = static_cast<uint32_t>(dst); o.d[1] = static_cast<uint32_t>(dst >> 32);
  o.d[2] = found; o.d[3] = left - 1;
  o.d[4] = 0; o.d[5] = 0;
}

namespace kcw {

constexpr uint32_t kStageWords = 2304;           // 384 out-neighbours; with the 256-entry task stack the group's LDS is full
constexpr uint32_t kRowWords = kStageWords / 2;  // rows under construction; the other half holds N+(u)
constexpr uint32_t kChunks = 4;                  // 64-element chunks of a concatenated stream in flight

struct Lds {
  union {
    uint64_t stage[kStageWords];  // edges and branches: the vertex's matrix
    struct {
      int32_t nu[2 * (kStageWords - kRowWords)];  // rows: N+(u) (vertices in place: theirs one after another)
      uint64_t row[kRowWords];                    // rows under construction
    };
  };
  uint64_t A[kWave];    // matrix the counting uses
  uint64_t B[kWave];    // vertices in place: undirected rows (pivoting)
  uint64_t acc[kWave];  // vertices in place: cliques per vertex
  uint32_t list[kWave];  // edges and branches: the candidates; vertices in place: words moved
  uint32_t seg[kWave], vtx[kWave];  // vertices in place: first row of a row's vertex, the vertex's lane
  uint32_t mark[kChunks * kWave];
};
static_assert(2 * (kStageWords - kRowWords) >= kcs::kMaxW * 64, "N+(u) fits");
static_assert(kRowWords >= kcs::kMaxW, "a row fits");

GTAP_DEV uint64_t shfl64(uint64_t x, uint32_t k) {
  const uint32_t lo = static_cast<uint32_t>(__shfl(static_cast<int>(static_cast<uint32_t>(x)), static_cast<int>(k), 64));
  const uint32_t hi = static_cast<uint32_t>(__shfl(static_cast<int>(static_cast<uint32_t>(x >> 32)), static_cast<int>(k), 64));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}
GTAP_DEV uint32_t shfl32(uint32_t x, uint32_t k) {
  return static_cast<uint32_t>(__shfl(static_cast<int>(x), static_cast<int>(k), 64));
}
GTAP_DEV uint32_t lane32(uint32_t x, int k) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), k));
}
GTAP_DEV uint32_t wave_sum(uint32_t x) { return lane32(wave_inclusive_sum(x), 63); }
GTAP_DEV void lds_or(uint64_t *p, uint64_t v) {
  __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
GTAP_DEV void lds_add(uint64_t *p, uint64_t v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Position of the j-th set bit of x (j below its population count).
GTAP_DEV uint32_t select64(uint64_t x, uint32_t j) {
  uint32_t pos = 0;
  uint32_t t = __popc(static_cast<uint32_t>(x));
  uint32_t v = static_cast<uint32_t>(x);
  if (j >= t) {
    j -= t;
    pos = 32;
    v = static_cast<uint32_t>(x >> 32);
  }
#pragma unroll
  for (uint32_t w = 16; w >= 1; w >>= 1) {
    t = __popc(v & ((1u << w) - 1u));
    if (j >= t) {
      j -= t;
      pos += w;
      v >>= w;
    }
  }
  return pos;
}

// The lane that owns each of the positions c0 + q * 64 + lane of a
// concatenation of lists (this lane's: [pre, pre + len)): marks at the lists'
// first positions, carried on by prefix maxima.  All lanes call it.
GTAP_DEV void chunk_owners(uint32_t *mark, uint32_t pre, uint32_t len, uint32_t c0, uint32_t (&own)[kChunks]) {
  const uint32_t ln = lane_id();
#pragma unroll
  for (uint32_t q = 0; q < kChunks; ++q) mark[q * kWave + ln] = 0;
  wave_sync();
  if (len > 0 && pre < c0 + kChunks * kWave && pre + len > c0) mark[pre > c0 ? pre - c0 : 0u] = ln + 1;
  wave_sync();
  uint32_t m[kChunks];
#pragma unroll
  for (uint32_t q = 0; q < kChunks; ++q) m[q] = wave_inclusive_max(mark[q * kWave + ln]);
  uint32_t carry = 0;
#pragma unroll
  for (uint32_t q = 0; q < kChunks; ++q) {
    m[q] = m[q] ? m[q] : carry;
    carry = lane32(m[q], 63);
    own[q] = m[q] ? m[q] - 1 : 0;
  }
  wave_sync();
}

// Walk the concatenation of the lanes' out-lists col[beg, beg + len) and
// search every element in the ascending list nu[lo, lo + n) (LDS; n <=
// `longest`, wave-uniform): hit(owner lane, index) for each element found.
// All lanes call it.
template <class Hit>
GTAP_DEV void scan_lists(uint32_t *mark, const int32_t *__restrict__ col, uint32_t beg, uint32_t len, const int32_t *nu,
                         uint32_t lo, uint32_t n, uint32_t longest, Hit hit) {
  const uint32_t ln = lane_id();
  uint32_t total = 0;
  const uint32_t pre = wave_exclusive_scan(len, &total);
  uint32_t top = 1;
  while (top * 2 <= longest) top *= 2;
  const uint32_t shift = beg - pre;  // position in col of concatenated position p: p + shift
  for (uint32_t c0 = 0; c0 < total; c0 += kChunks * kWave) {
    uint32_t own[kChunks], at[kChunks], end[kChunks];
    int32_t y[kChunks];
    chunk_owners(mark, pre, len, c0, own);
#pragma unroll
    for (uint32_t q = 0; q < kChunks; ++q) {
      const uint32_t pos = c0 + q * kWave + ln;
      const uint32_t sh = shfl32(shift, own[q]);
      at[q] = shfl32(lo, own[q]);
      end[q] = at[q] + shfl32(n, own[q]);
      y[q] = 0;
      if (pos < total) y[q] = col[pos + sh];
      else end[q] = at[q];  // an empty range: nothing found
    }
    // at: first index not below y (halving steps, the chunks side by side)
    for (uint32_t step = top; step >= 1; step >>= 1) {
#pragma unroll
      for (uint32_t q = 0; q < kChunks; ++q) {
        const uint32_t t = at[q] + step;
        const bool in = t <= end[q];
        const int32_t v = nu[in ? t - 1 : 0u];
        if (in && v < y[q]) at[q] = t;
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kChunks; ++q) {
      const bool in = at[q] < end[q];
      const int32_t v = nu[in ? at[q] : 0u];
      if (in && v == y[q]) hit(own[q], at[q]);
    }
  }
}

// The other way round: each lane's `cnt` needles nu[first, first + cnt) (LDS),
// all lanes' concatenated, are searched in the needle's own lane's out-list
// col[beg, beg + len).  hit(owner lane, index of the needle).
template <class Hit>
GTAP_DEV void scan_needles(uint32_t *mark, const int32_t *__restrict__ col, uint32_t beg, uint32_t len,
                           const int32_t *nu, uint32_t first, uint32_t cnt, Hit hit) {
  const uint32_t ln = lane_id();
  uint32_t total = 0;
  const uint32_t pre = wave_exclusive_scan(cnt, &total);
  const uint32_t longest = lane32(wave_inclusive_max(cnt > 0 ? len : 0u), 63);
  uint32_t top = 1;
  while (top * 2 <= longest) top *= 2;
  const uint32_t shift = first - pre;
  for (uint32_t c0 = 0; c0 < total; c0 += kChunks * kWave) {
    uint32_t own[kChunks], at[kChunks], end[kChunks], idx[kChunks];
    int32_t y[kChunks], seen[kChunks];
    chunk_owners(mark, pre, cnt, c0, own);
#pragma unroll
    for (uint32_t q = 0; q < kChunks; ++q) {
      const uint32_t pos = c0 + q * kWave + ln;
      idx[q] = pos + shfl32(shift, own[q]);
      at[q] = shfl32(beg, own[q]);
      end[q] = at[q] + shfl32(len, own[q]);
      y[q] = 0;
      seen[q] = -1;  // no vertex
      if (pos < total) y[q] = nu[idx[q]];
      else end[q] = at[q];
    }
    // at: one past the last element not above y; seen: the largest element
    // compared that was not above it
    for (uint32_t step = top; step >= 1; step >>= 1) {
      int32_t v[kChunks];
#pragma unroll
      for (uint32_t q = 0; q < kChunks; ++q) {
        const uint32_t t = at[q] + step;
        v[q] = t <= end[q] ? col[t - 1] : 0x7FFFFFFF;
      }
#pragma unroll
      for (uint32_t q = 0; q < kChunks; ++q)
        if (v[q] <= y[q] && at[q] + step <= end[q]) {
          at[q] += step;
          seen[q] = v[q];
        }
    }
#pragma unroll
    for (uint32_t q = 0; q < kChunks; ++q)
      if (seen[q] == y[q]) hit(own[q], idx[q]);
  }
}

// m-cliques (m >= 1) of the DAG with one-word rows A on the set T.
GTAP_DEV int64_t inner_cliques(const uint64_t *A, uint64_t T, uint32_t m) {
  if (m == 1) return __popcll(T);
  if (static_cast<uint32_t>(__popcll(T)) < m) return 0;
  int64_t total = 0;
  if (m == 2) {
    for (uint64_t t = T; t; t &= t - 1) total += __popcll(T & A[__builtin_ctzll(t)]);
    return total;
  }
  if (m == 3) {
    for (uint64_t t = T; t; t &= t - 1) {
      const uint64_t T2 = T & A[__builtin_ctzll(t)];
      for (uint64_t s = T2; s; s &= s - 1) total += __popcll(T2 & A[__builtin_ctzll(s)]);
    }
    return total;
  }
  return kcs::dag_count(A, T, m);
}

// For every lane's row r and every member b of it: m-cliques of r /\ A[base + b]
// (A indexed from the lane's base; m >= 1, wave-uniform).  The pairs are dealt
// to the lanes; add(owner lane, count) receives each count.
template <class Add>
GTAP_DEV void count_pairs(const uint64_t *A, uint32_t *mark, uint64_t r, uint32_t base, uint32_t m, Add add) {
  const uint32_t ln = lane_id();
  const uint32_t nb = __popcll(r);
  uint32_t total = 0;
  const uint32_t off = wave_exclusive_scan(nb, &total);
  uint32_t carry = 0;
  for (uint32_t e0 = 0; e0 < total; e0 += kWave) {
    const uint32_t own = chunk_owner(mark, nb, off, e0, carry);
    const uint64_t ro = shfl64(r, own);
    const uint32_t bo = shfl32(base, own), j = e0 + ln - shfl32(off, own);
    if (e0 + ln < total) {
      const uint64_t T = ro & A[bo + select64(ro, j)];
      const int64_t v = inner_cliques(A + bo, T, m);
      if (v) add(own, v);
    }
  }
}

// A job's arguments and the matrix of the vertex the wavefront is at,
// wave-uniform.
struct Job {
  const int32_t *rp;
  const int32_t *col;
  uint64_t *mat;  // n+1 vertex offsets, then the bit matrices
  uint32_t n, kk, thr;
  bool pivot;
};
GTAP_DEV Job load_job(const JobSlot *J) {
  uint64_t a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = co_ld64(&J->a[i]);
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = uniform64(a[i]);
  return Job{reinterpret_cast<const int32_t *>(a[0]), reinterpret_cast<const int32_t *>(a[1]),
             reinterpret_cast<uint64_t *>(a[7]), static_cast<uint32_t>(a[2]), static_cast<uint32_t>(a[3]) - 2,
             static_cast<uint32_t>(a[6] & 0xFFu), ((a[6] >> 8) & 1u) != 0};
}
struct Mat {
  uint64_t *D;     // row i: the members of N+(u) that are out-neighbours of its i-th member
  uint64_t *rows;  // what the search uses: D, for pivoting U (D or its transpose)
  uint32_t d, W;
};
GTAP_DEV Mat load_mat(const Job &J, uint32_t u) {
  const uint32_t r0 = static_cast<uint32_t>(J.rp[u]), r1 = static_cast<uint32_t>(J.rp[u + 1]);
  const uint64_t off = co_ld64(J.mat + u);
  const uint32_t d = uniform(r1 - r0), W = (d + 63) / 64;
  uint64_t *D = J.mat + (J.n + 1) + uniform64(off);
  return Mat{D, J.pivot ? D + static_cast<size_t>(d) * W : D, d, W};
}

// ---- rows -------------------------------------------------------------------
// Row tasks of the lanes in `todo` (lane k: row i[k] of vertex u[k]).  words:
// each lane's count of task data moved.
GTAP_DEV void run_rows(Lds &S, const JobSlot *jobs, uint64_t todo, uint32_t job, uint32_t u, uint32_t i,
                       uint32_t &words) {
  const uint32_t ln = lane_id();
  uint32_t cur_job = kNone;
  Job J{};
  while (todo) {
    const int k = __builtin_ctzll(todo);
    const uint32_t kj = lane32(job, k), ku = lane32(u, k);
    if (kj != cur_job) {
      J = load_job(jobs + kj);
      cur_job = kj;
    }
    const Mat M = load_mat(J, ku);
    const uint32_t s0 = uniform(static_cast<uint32_t>(J.rp[ku]));
    // the siblings among the lanes, as many as the row buffer holds
    const bool same = ((todo >> ln) & 1u) != 0 && job == kj && u == ku;
    uint64_t g = ballot(same);
    uint32_t r = rank_below(g);
    const bool mine = same && (r + 1) * M.W <= kRowWords;
    g = ballot(mine);
    todo &= ~g;
    int32_t *nu = S.nu;
    uint64_t *row = S.row;
    wave_sync();
    for (uint32_t t = ln; t < M.d; t += kWave) nu[t] = J.col[s0 + t];
    for (uint32_t t = ln; t < static_cast<uint32_t>(__popcll(g)) * M.W; t += kWave) row[t] = 0;
    wave_sync();
    uint32_t beg = 0, len = 0;
    bool before = false;  // N+(x) begins before x
    if (mine) {
      const int32_t x = nu[i];
      beg = static_cast<uint32_t>(J.rp[x]);
      len = static_cast<uint32_t>(J.rp[x + 1]) - beg;
      if (len > 0) before = J.col[beg] < x;
      words = 4 + M.d + len + (J.pivot ? 4 : 2) * M.W;  // row bounds, both lists, the row (and U's) written
    }
    uint64_t *U = M.rows;
    const uint32_t W = M.W;
    const bool pivot = J.pivot;
    auto hit = [&](uint32_t own, uint32_t j) {
      const uint32_t ro = static_cast<uint32_t>(__popcll(g & ((1ull << own) - 1ull)));
      lds_or(row + ro * W + (j >> 6), 1ull << (j & 63));
    };
    // the shorter of N+(x) and the members that can be in it is searched in the other
    const uint32_t first = before ? 0u : i + 1, rest = mine ? M.d - first : 0u;
    const bool walk = len < rest;
    if (ballot(walk) != 0ull) scan_lists(S.mark, J.col, beg, walk ? len : 0u, nu, 0u, M.d, M.d, hit);
    scan_needles(S.mark, J.col, beg, len, nu, first, walk ? 0u : rest, hit);
    wave_sync();
    if (mine) {
      for (uint32_t w = 0; w < W; ++w) {
        uint64_t v = row[r * W + w];
        co_st64(M.D + static_cast<size_t>(i) * W + w, v);
        if (pivot && v) {
          fetch_or_relaxed(U + static_cast<size_t>(i) * W + w, v);
          for (; v; v &= v - 1)
            fetch_or_relaxed(U + static_cast<size_t>(w * 64 + __builtin_ctzll(v)) * W + (i >> 6),
                             static_cast<uint64_t>(1) << (i & 63));
        }
      }
    }
    wave_sync();
  }
}

// Clear U of each lane's vertex in `todo` (pivoting; its rows are ORed in by
// the row tasks, which run after this wavefront's stores completed).
GTAP_DEV void clear_mats(const JobSlot *jobs, uint64_t todo, uint32_t job, uint32_t u) {
  while (todo) {
    const int k = __builtin_ctzll(todo);
    todo &= todo - 1;
    const Job J = load_job(jobs + lane32(job, k));
    const Mat M = load_mat(J, lane32(u, k));
    for (uint32_t t = lane_id(); t < M.d * M.W; t += kWave) co_st64(M.rows + t, 0ull);
  }
  drain();
}

// ---- vertices in place ----------------------------------------------------------
// Vertices with at most 64 out-neighbours (lane k: vertex with deg[k]
// out-neighbours from col[s0[k]]): as many neighbouring lanes' vertices at a
// time as have 64 out-neighbours together, one row per lane.
GTAP_DEV void run_vertices(Lds &S, const JobSlot *jobs, uint64_t todo, uint32_t job, uint32_t s0, uint32_t deg,
                           int64_t &value, uint32_t &words) {
  const uint32_t ln = lane_id();
  uint32_t cur_job = kNone;
  Job J{};
  int32_t *nu = S.nu;
  while (todo) {
    const int k = __builtin_ctzll(todo);
    const uint32_t kj = lane32(job, k);
    if (kj != cur_job) {
      J = load_job(jobs + kj);
      cur_job = kj;
    }
    const bool same = ((todo >> ln) & 1u) != 0 && job == kj;
    const uint32_t dl = same ? deg : 0u;
    const uint32_t incl = wave_inclusive_sum(dl);
    const bool mine = same && incl <= kWave;
    const uint64_t g = ballot(mine);
    todo &= ~g;
    const uint32_t pre = incl - dl;  // first row of this lane's vertex
    const uint32_t rows = lane32(incl, 63 - __builtin_clzll(g));
    wave_sync();
    S.mark[ln] = 0;
    S.A[ln] = 0;
    S.B[ln] = 0;
    S.acc[ln] = 0;
    S.list[ln] = 0;
    wave_sync();
    if (mine) S.mark[pre] = ln + 1;
    wave_sync();
    const uint32_t m = wave_inclusive_max(S.mark[ln]);
    const uint32_t own = m ? m - 1 : 0u;  // vertex of row ln
    const bool row = ln < rows;
    const uint32_t seg = shfl32(pre, own), dv = shfl32(dl, own), at = shfl32(s0, own) + ln - seg;
    wave_sync();
    S.seg[ln] = seg;
    S.vtx[ln] = own;
    uint32_t beg = 0, len = 0;
    bool before = false;
    if (row) {
      const int32_t x = J.col[at];
      nu[ln] = x;
      beg = static_cast<uint32_t>(J.rp[x]);
      len = static_cast<uint32_t>(J.rp[x + 1]) - beg;
      if (len > 0) before = J.col[beg] < x;
      __hip_atomic_fetch_add(&S.list[own], 2 + len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    wave_sync();
    const bool pivot = J.pivot;
    auto hit = [&](uint32_t r, uint32_t j) {
      const uint32_t sg = S.seg[r];
      lds_or(&S.A[r], 1ull << (j - sg));
      if (pivot) {
        lds_or(&S.B[r], 1ull << (j - sg));
        lds_or(&S.B[j], 1ull << (r - sg));
      }
    };
    const uint32_t first = before ? seg : ln + 1, rest = row ? seg + dv - first : 0u;
    const bool walk = len < rest;
    if (ballot(walk) != 0ull) scan_lists(S.mark, J.col, beg, walk ? len : 0u, nu, seg, row ? dv : 0u, kWave, hit);
    scan_needles(S.mark, J.col, beg, len, nu, first, walk ? 0u : rest, hit);
    wave_sync();
    uint64_t a = row ? S.A[ln] : 0ull;
    if (static_cast<uint32_t>(__popcll(a)) < J.kk) a = 0ull;
    if (!pivot) {
      count_pairs(S.A, S.mark, a, seg, J.kk - 1, [&](uint32_t r, int64_t v) { lds_add(&S.acc[S.vtx[r]], static_cast<uint64_t>(v)); });
    } else if (a) {
      const int64_t v = kcs::sct_count(S.B + seg, a, 0, 0, J.kk);
      if (v) lds_add(&S.acc[own], static_cast<uint64_t>(v));
    }
    wave_sync();
    if (mine) {
      value = static_cast<int64_t>(S.acc[ln]);
      words += deg + S.list[ln];
    }
    wave_sync();
  }
}

// ---- sets of W words in registers, rows staged in LDS -------------------------------
template <uint32_t W>
GTAP_DEV uint32_t count_w(const uint64_t (&x)[W]) {
  uint32_t n = 0;
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) n += __popcll(x[w]);
  return n;
}
// The j-th member (j below the count).
template <uint32_t W>
GTAP_DEV uint32_t select_w(const uint64_t (&x)[W], uint32_t j) {
  uint64_t cur = x[0];
  uint32_t at = 0;
#pragma unroll
  for (uint32_t w = 1; w < W; ++w) {
    const uint32_t n = __popcll(cur);
    if (at == (w - 1) * 64 && j >= n) {
      j -= n;
      cur = x[w];
      at = w * 64;
    }
  }
  return at + select64(cur, j);
}
// Take the lowest member out of the set; false when it is empty.
template <uint32_t W>
GTAP_DEV bool take_w(uint64_t (&x)[W], uint32_t &y) {
  bool got = false;
#pragma unroll
  for (uint32_t w = 0; w < W; ++w)
    if (!got && x[w] != 0ull) {
      y = w * 64 + __builtin_ctzll(x[w]);
      x[w] &= x[w] - 1;
      got = true;
    }
  return got;
}
template <uint32_t W>
GTAP_DEV void and_row(const uint64_t *rows, const uint64_t (&x)[W], uint32_t y, uint64_t (&out)[W]) {
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) out[w] = x[w] & rows[y * W + w];
}
// m-cliques (1 <= m <= 3) of the DAG with the given rows on the set T.
template <uint32_t W>
GTAP_DEV uint32_t inner_w(const uint64_t *rows, const uint64_t (&T)[W], uint32_t m) {
  const uint32_t c = count_w<W>(T);
  if (m == 1) return c;
  if (c < m) return 0;
  uint32_t total = 0, y = 0, z = 0;
  uint64_t r[W], T2[W], T3[W];
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) r[w] = T[w];
  while (take_w<W>(r, y)) {
    and_row<W>(rows, T, y, T2);
    const uint32_t n = count_w<W>(T2);
    if (m == 2) {
      total += n;
    } else if (n >= 2) {
      uint64_t r2[W];
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) r2[w] = T2[w];
      while (take_w<W>(r2, z)) {
        and_row<W>(rows, T2, z, T3);
        total += count_w<W>(T3);
      }
    }
  }
  return total;
}

// Orientation: the edges, heavy edges' roots and branches of one vertex (the
// lanes in `g`), rows of W <= 6 words staged in LDS, cliques of at most five
// members inside an edge's candidates.  Every lane forms its own task's
// candidate set; then the (task, candidate) pairs of all the tasks are dealt to
// the lanes, and of those whose row keeps enough candidates the
// (task, candidate, candidate) triples, each finished by one lane.
template <uint32_t W>
GTAP_DEV void run_sets(const Params &p, Lds &S, const Job &J, uint64_t g, uint32_t tid, Outcome &o) {
  const uint32_t ln = lane_id();
  const bool mine = ((g >> ln) & 1u) != 0;
  const bool node = mine && o.kind == TK_KS_NODE, heavy = mine && o.kind == TK_KS_HEAVY;
  const uint64_t *rows = S.stage;
  uint64_t s[W];
  uint32_t l = J.kk, words = 4 + 2 * W;  // row bounds, matrix offset, the edge's row
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) s[w] = 0;
  if (mine) {
    const uint32_t i = o.d[1];
    if (node) {
      const uint64_t *pb = reinterpret_cast<const uint64_t *>(frame_ptr(p, o.parent) + FW_BUF);
      const uint64_t meta = co_ld64(pb);
      uint64_t P[W];
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) P[w] = co_ld64(pb + 1 + w);
      l = static_cast<uint32_t>(meta & 0xFFFFu) - 1;
      and_row<W>(rows, P, select_w<W>(P, i), s);
      words = 6 + 4 * W;  // row bounds, matrix offset, node meta and set, one row
    } else {
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) s[w] = rows[i * W + w];
    }
  }
  const uint32_t c = count_w<W>(s);
  const bool some = mine && !heavy && l > 1 && c >= l;
  const bool in_place = some && (l == 2 || c <= J.thr);
  const bool split = heavy || (some && !in_place && node);
  if (heavy) words += 2 + 2 * W;  // node state
  else if (in_place || split) words += 2 * W * c;  // the candidates' rows
  S.acc[ln] = 0;
  wave_sync();
  // triples waiting to be finished, on lanes [0, np): about one in ten keeps
  // enough candidates, so they are gathered until the lanes are full
  uint64_t wt[W];
  uint32_t wm = 1, wtask = 0, np = 0;
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) wt[w] = 0;
  auto finish = [&]() {
    if (ln < np) {
      const uint32_t v = inner_w<W>(rows, wt, wm);
      if (v) lds_add(&S.acc[wtask], v);
    }
    np = 0;
  };
  uint32_t total = 0;
  const uint32_t n0 = in_place ? c : 0u;
  const uint32_t off = wave_exclusive_scan(n0, &total);
  uint32_t carry = 0;
  for (uint32_t e0 = 0; e0 < total; e0 += kWave) {
    const uint32_t own = chunk_owner(S.mark, n0, off, e0, carry);
    uint64_t so[W], t[W];
#pragma unroll
    for (uint32_t w = 0; w < W; ++w) so[w] = shfl64(s[w], own);
    const uint32_t lo = shfl32(l, own), j = e0 + ln - shfl32(off, own);
    const bool act = e0 + ln < total;
    and_row<W>(rows, so, act ? select_w<W>(so, j) : 0u, t);
    const uint32_t n = act ? count_w<W>(t) : 0u;
    if (lo == 2 && n > 0) lds_add(&S.acc[own], n);
    const uint32_t n1 = lo > 2 && n >= lo - 1 ? n : 0u;
    uint32_t total1 = 0, carry1 = 0;
    const uint32_t off1 = wave_exclusive_scan(n1, &total1);
    for (uint32_t f0 = 0; f0 < total1; f0 += kWave) {
      const uint32_t own1 = chunk_owner(S.mark, n1, off1, f0, carry1);
      uint64_t to[W], t1[W];
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) to[w] = shfl64(t[w], own1);
      const uint32_t m = shfl32(lo, own1) - 2, task = shfl32(own, own1), j1 = f0 + ln - shfl32(off1, own1);
      const bool act1 = f0 + ln < total1;
      and_row<W>(rows, to, act1 ? select_w<W>(to, j1) : 0u, t1);
      const uint32_t c1 = act1 ? count_w<W>(t1) : 0u;
      if (m == 1 && c1 > 0) lds_add(&S.acc[task], c1);
      const uint64_t keep = ballot(m > 1 && c1 >= m);
      const uint32_t nk = static_cast<uint32_t>(__popcll(keep));
      if (nk == 0) continue;
      if (np + nk > kWave) finish();
      const bool take = ln >= np && ln < np + nk;
      const uint32_t from = take ? select64(keep, ln - np) : ln;
      const uint32_t mk = shfl32(m, from), tk = shfl32(task, from);
      wm = take ? mk : wm;
      wtask = take ? tk : wtask;
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) {
        const uint64_t x = shfl64(t1[w], from);
        wt[w] = take ? x : wt[w];
      }
      np += nk;
    }
  }
  finish();
  wave_sync();
  if (!mine) return;
  o.words = words;
  if (in_place) o.value = static_cast<int64_t>(S.acc[ln]);
  else if (l == 1 && !heavy) o.value = c;
  if (split) {  // node state into the task's frame; one child per candidate
    uint64_t *b = reinterpret_cast<uint64_t *>(frame_ptr(p, tid) + FW_BUF);
    co_st64(b, static_cast<uint64_t>(l));
#pragma unroll
    for (uint32_t w = 0; w < W; ++w) co_st64(b + 1 + w, s[w]);
    o.type = OUT_FORK;
    o.nchild = c;
    o.ckind = TK_KS_NODE;
    o.big = l - 1 >= 3 ? 1u : 0u;  // children that may split keep state in a big frame
    o.d[1] = 0;
  } else if (some && !in_place) {  // an edge with many candidates: one task takes the search over
    o.type = OUT_FORK;
    o.nchild = 1;
    o.ckind = TK_KS_HEAVY;
    o.big = 1;
  }
}

// ---- edges, heavy edges' roots and branches -----------------------------------------
// The tasks of the lanes in `todo` (o.d: vertex, index).  Sets o.value, or the
// fork of a task that splits.  Tasks that run_sets cannot take (pivoting,
// matrices too large for LDS, cliques of six or more members inside the
// candidates) run one after another, the candidate set one word per lane (lane
// w: word w).
GTAP_DEV void run_search(const Params &p, Lds &S, uint64_t todo, uint32_t tid, Outcome &o) {
  const uint32_t ln = lane_id();
  uint32_t cur_job = kNone, cur_u = kNone, cur_par = kNone;
  bool staged = false;
  Job J{};
  Mat M{};
  uint64_t meta = 0, Pw = 0, Rw = 0;  // node state of the current branches' parent
  drain();  // node state this wavefront wrote in its last iteration
  while (todo) {
    const int k = __builtin_ctzll(todo);
    todo &= todo - 1;
    const uint32_t kj = lane32(o.job, k), ku = lane32(o.d[0], k), ki = lane32(o.d[1], k);
    const uint32_t kind = lane32(o.kind, k);
    if (kj != cur_job) {
      J = load_job(p.jobs + kj);
      cur_job = kj;
      cur_u = cur_par = kNone;
      if (J.pivot || J.kk > 5) {
        // the job's edges with too few candidates, by their own lanes (run_sets
        // looks at its rows itself): where thresholds are small half of all
        // these tasks end so (30,000 vertices, threshold 16, pivoting: k = 6 8.4
        // -> 7.7 ms; run one after another they made such calls slower than a
        // lane for each task, 4.9 and 7.3 ms at k = 4 and 6)
        bool done = false;
        if (((1ull << k | todo) >> ln & 1u) != 0 && o.job == kj && o.kind == TK_KS_EDGE) {
          const uint32_t u = o.d[0], W = (static_cast<uint32_t>(J.rp[u + 1] - J.rp[u]) + 63) / 64;
          const uint64_t *row = J.mat + (J.n + 1) + co_ld64(J.mat + u) + static_cast<size_t>(o.d[1]) * W;
          uint32_t c = 0;
          for (uint32_t w = 0; w < W; ++w) c += __popcll(co_ld64(row + w));
          done = c < J.kk;
          if (done) {
            o.value = 0;
            o.words = 4 + 2 * W;  // row bounds, matrix offset, the edge's row
          }
        }
        const uint64_t m = ballot(done);
        todo &= ~m;
        if ((m >> k) & 1u) continue;
      }
    }
    if (ku != cur_u) {
      M = load_mat(J, ku);
      cur_u = ku;
      const uint32_t nw = M.d * M.W;
      staged = nw <= kStageWords;
      if (staged) {
        wave_sync();
        for (uint32_t t = ln; t < nw; t += 4 * kWave) {
          uint64_t v[4];
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q) v[q] = t + q * kWave < nw ? co_ld64(M.rows + t + q * kWave) : 0ull;
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q)
            if (t + q * kWave < nw) S.stage[t + q * kWave] = v[q];
        }
        wave_sync();
      }
    }
    if (staged && !J.pivot && M.W <= 6 && J.kk <= 5) {
      const uint64_t g = ballot(((1ull << k | todo) >> ln & 1u) != 0 && o.job == kj && o.d[0] == ku);
      todo &= ~g;
      switch (M.W) {
        case 1: run_sets<1>(p, S, J, g, tid, o); break;
        case 2: run_sets<2>(p, S, J, g, tid, o); break;
        case 3: run_sets<3>(p, S, J, g, tid, o); break;
        case 4: run_sets<4>(p, S, J, g, tid, o); break;
        case 5: run_sets<5>(p, S, J, g, tid, o); break;
        default: run_sets<6>(p, S, J, g, tid, o); break;
      }
      continue;
    }
    const uint32_t W = M.W;
    auto word = [&](uint32_t y, uint32_t w) -> uint64_t {
      return staged ? S.stage[y * W + w] : co_ld64(M.rows + static_cast<size_t>(y) * W + w);
    };
    auto word_of = [&](uint64_t x, uint32_t w) -> uint64_t { return readlane64(x, static_cast<int>(w)); };
    // the j-th member of a set held one word per lane
    auto member = [&](uint64_t x, uint32_t j) -> uint32_t {
      const uint32_t n = __popcll(x), incl = wave_inclusive_sum(n), pre = incl - n;
      const uint64_t m = ballot(j >= pre && j < incl);
      const int w = m ? __builtin_ctzll(m) : 0;
      return static_cast<uint32_t>(w) * 64 + lane32(select64(x, j >= pre ? j - pre : 0u), w);
    };
    uint64_t s = 0;
    uint32_t l = J.kk, h = 0, q = 0, words = 4 + 2 * W;  // row bounds, matrix offset, the edge's row
    const bool node = kind == TK_KS_NODE;
    if (node) {
      const uint32_t par = lane32(o.parent, k);
      if (par != cur_par) {
        const uint64_t *pb = reinterpret_cast<const uint64_t *>(frame_ptr(p, par) + FW_BUF);
        meta = co_ld64(pb);
        Pw = ln < W ? co_ld64(pb + 1 + ln) : 0ull;
        Rw = J.pivot && ln < W ? co_ld64(pb + 1 + W + ln) : 0ull;
        meta = uniform64(meta);
        cur_par = par;
      }
      words = 6 + 4 * W;  // row bounds, matrix offset, node meta and set, one row
      if (!J.pivot) {
        l = static_cast<uint32_t>(meta & 0xFFFFu) - 1;
        const uint32_t x = member(Pw, ki);
        if (ln < W) s = Pw & word(x, ln);
      } else {
        h = static_cast<uint32_t>(meta & 0xFFFFu);
        q = static_cast<uint32_t>((meta >> 16) & 0xFFFFu);
        const uint32_t piv = static_cast<uint32_t>(meta >> 32);
        if (ki == 0) {  // the pivot branch
          if (ln < W) s = Pw & word(piv, ln);
          q += 1;
        } else {  // the (ki-1)-th non-neighbour of the pivot, held
          const uint32_t x = member(Rw, ki - 1);
          const uint64_t before = ln < (x >> 6) ? Rw : ln == (x >> 6) ? (Rw & kcs::low_mask(x & 63)) : 0ull;
          if (ln < W) s = Pw & ~before & word(x, ln);
          if (ln == (piv >> 6)) s &= ~(1ull << (piv & 63));
          h += 1;
        }
      }
    } else if (ln < W) {
      s = staged && !J.pivot ? S.stage[ki * W + ln] : co_ld64(M.D + static_cast<size_t>(ki) * W + ln);
    }
    const uint32_t c = wave_sum(__popcll(s));
    // what to do with the candidate set: finished (val), counted in place or split
    int64_t val = 0;
    enum { kDone, kPairs, kCount, kSplit, kHeavy } act = kDone;
    uint32_t few = 0;  // pivoting, in place: members still to be chosen, when at most two
    if (kind == TK_KS_HEAVY) {
      act = kSplit;
      words += J.pivot ? 2 * W * (c + 1) + 2 + 4 * W : 2 + 2 * W;  // pivot rows; node state
    } else if (J.pivot) {
      if (node && h == J.kk) val = 1;
      else if (node && c == 0) val = kcs::binom(q, J.kk - h);
      else if (c + q >= J.kk - h) act = c <= J.thr ? kCount : node ? kSplit : kHeavy;
      if (act == kCount || act == kSplit) words += 2 * W * (c + (node && ki != 0 ? 1 : 0));  // the candidates' rows (and R)
      if (act == kCount && J.kk - h <= 2) {  // from the candidates and the q pivots, which all are neighbours (k = 4: 5.6 -> 1.6 ms)
        few = J.kk - h;
        act = few == 2 ? kPairs : kDone;
        if (few == 1) val = c + q;
      }
    } else {
      if (l == 1) val = c;
      else if (c >= l) act = l == 2 ? kPairs : c <= J.thr ? kCount : node ? kSplit : kHeavy;
      if (act != kDone && act != kHeavy) words += 2 * W * c;  // the candidates' rows
    }
    uint32_t nchild = 0;
    if (act == kPairs) {  // directed edges inside the set
      uint32_t e = 0;
      for (uint32_t w = 0; w < W; ++w) {
        if ((word_of(s, w) >> ln) & 1u)
          for (uint32_t v = 0; v < W; ++v) e += __popcll(word(w * 64 + ln, v) & word_of(s, v));
      }
      val = wave_sum(e);
      if (few == 2) val = val / 2 + static_cast<int64_t>(c) * q + static_cast<int64_t>(q) * (q - 1) / 2;  // rows hold both directions
    } else if (act == kCount) {
      // the candidates, one per lane
      wave_sync();
      uint32_t pre = 0;
      for (uint32_t w = 0; w < W; ++w) {
        const uint64_t sw = word_of(s, w);
        if ((sw >> ln) & 1u) S.list[pre + rank_below(sw)] = w * 64 + ln;
        pre += static_cast<uint32_t>(__popcll(sw));
      }
      wave_sync();
      const uint32_t y = ln < c ? S.list[ln] : 0u;
      bool any = true;
      if (!J.pivot) {  // a clique's first member has l - 1 of the candidates as out-neighbours
        uint32_t n = 0;
        for (uint32_t w = 0; w < W; ++w) n += __popcll(word(y, w) & word_of(s, w));
        any = ballot(ln < c && n >= l - 1) != 0ull;
      }
      if (any) {
        // column b: the candidates that have the b-th one in their row
        uint64_t col = 0;
        uint32_t b = 0;
        for (uint32_t w = 0; w < W; ++w) {
          const uint64_t sw = word_of(s, w);
          if (sw == 0ull) continue;
          const uint64_t r = ln < c ? word(y, w) : 0ull;
          for (uint64_t t = sw; t; t &= t - 1, ++b) {
            const uint64_t m = ballot(((r >> __builtin_ctzll(t)) & 1u) != 0);
            if (ln == b) col = m;
          }
        }
        S.A[ln] = col;
        wave_sync();
        int64_t v = 0;
        if (!J.pivot) {
          count_pairs(S.A, S.mark, col, 0u, l - 2, [&](uint32_t, int64_t x) { v += x; });
        } else {
          // the root's branches: the pivot (most neighbours, lowest on ties), then its non-neighbours
          const uint32_t key = ln < c ? ((static_cast<uint32_t>(__popcll(col)) + 1) << 6) | (63 - ln) : 0u;
          const uint32_t piv = 63 - (lane32(wave_inclusive_max(key), 63) & 63u);
          const uint64_t all = kcs::low_mask(c) & ~(1ull << piv), near = readlane64(col, static_cast<int>(piv));
          const uint64_t far = all & ~near;
          if (ln <= static_cast<uint32_t>(__popcll(far))) {
            uint64_t P = near;
            if (ln > 0) {
              const uint32_t x = select64(far, ln - 1);
              P = all & ~(far & kcs::low_mask(x)) & S.A[x];
            }
            v = kcs::sct_count(S.A, P, ln > 0 ? h + 1 : h, ln > 0 ? q : q + 1, J.kk);
          }
        }
        val = static_cast<int64_t>(readlane64(wave_inclusive_sum64(static_cast<uint64_t>(v)), 63));
        wave_sync();
      }
    } else if (act == kSplit) {
      // node state into the task's frame; one child per branch
      uint64_t *b = reinterpret_cast<uint64_t *>(frame_ptr(p, lane32(tid, k)) + FW_BUF);
      uint64_t state = l;
      nchild = c;
      if (J.pivot) {
        uint32_t key = 0;  // most neighbours in the set, lowest on ties
        for (uint32_t w = 0; w < W; ++w) {
          if (!((word_of(s, w) >> ln) & 1u)) continue;
          uint32_t n = 0;
          for (uint32_t v = 0; v < W; ++v) n += __popcll(word(w * 64 + ln, v) & word_of(s, v));
          const uint32_t kw = ((n + 1) << 16) | (0xFFFFu - (w * 64 + ln));
          key = kw > key ? kw : key;
        }
        const uint32_t piv = 0xFFFFu - (lane32(wave_inclusive_max(key), 63) & 0xFFFFu);
        uint64_t r = ln < W ? s & ~word(piv, ln) : 0ull;
        if (ln == (piv >> 6)) r &= ~(1ull << (piv & 63));
        if (ln < W) co_st64(b + 1 + W + ln, r);
        nchild = 1 + wave_sum(__popcll(r));
        state = h | (static_cast<uint64_t>(q) << 16) | (static_cast<uint64_t>(piv) << 32);
      }
      if (ln < W) co_st64(b + 1 + ln, s);
      if (ln == 0) co_st64(b, state);
    }
    if (static_cast<int>(ln) == k) {
      o.value = val;
      o.words = words;
      if (act == kHeavy) {  // an edge with many candidates: one task takes the search over
        o.type = OUT_FORK;
        o.nchild = 1;
        o.ckind = TK_KS_HEAVY;
        o.big = 1;
      } else if (act == kSplit) {
        o.type = OUT_FORK;
        o.nchild = nchild;
        o.ckind = TK_KS_NODE;
        o.big = (J.pivot || l - 1 >= 3) ? 1u : 0u;  // children that may split keep state in a big frame
        o.d[1] = 0;
      }
    }
  }
}

}  // namespace kcw
}  // namespace gtap
