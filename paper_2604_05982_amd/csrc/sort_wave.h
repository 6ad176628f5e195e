// sort_wave.h -- Cilksort's serial sorts and merges, executed by the whole
// wavefront (Sec. 6.3).
//
// A lane whose task is a serial sort or a serial merge only describes it; the
// wavefront then takes the described ranges one after another, one key per
// lane (sort) or four (merge tile), so that every access to the keys is a
// 256-byte run instead of 64 lanes walking 64 runs a key at a time.  What
// bounded the lane-serial form was the chain of device-coherent loads (a
// merge of 256 keys is 256 dependent steps, each about a microsecond, on one
// lane).  100,003 keys on one queue: 6.7 ms in the kernel lane-serially, 3.1 ms
// this way (1.8 ms with tasks exposed early); 30 M keys on three queues: 26.6 ->
// 13.1 ms (9.2 ms with fresh frames claimed by one add).
//
// Both run as bitonic networks on registers: partners at lane distance 1..8
// come by DPP, 16 and 32 by the row-swap instructions, 64 and 128 are other
// registers, so a network touches no LDS.  A tile of 256 keys needs 8 rounds
// on 4 registers (about 80 instructions); the loads of the next tiles are
// issued before a network runs, which hides most of their latency.
//
// Sorts of at most 32 keys and merges of at most 64 would leave most of a
// register's lanes or of a tile empty, at the same number of rounds: with small
// cutoffs that was slower than the lane-serial form.  They share registers
// instead, 64 / W ranges of at most W keys side by side: 1 M keys with cutoffs
// 8 and 16: 10.3 ms lane-serially, 16.4 ms a range at a time, 8.2 ms this way;
// cutoffs 64 and 64: 12.7, 9.3 and 6.8 ms.  The bodies for that are compiled
// into a kernel of their own (kExtShort): in the other one they cost sorts with
// the default cutoffs 1 to 2 %.
#pragma once
#include "wave.h"

namespace gtap {
namespace cilk {

constexpr uint32_t kTileRegs = 4;
constexpr uint32_t kTile = kWave * kTileRegs;  // keys of one merge network
constexpr uint32_t kPad = 0xFFFFFFFFu;         // sorts last; never stored

// Bitonic compare-exchange at lane distance D: lanes with `low` keep the
// smaller key.  Every lane must be active.
template <int D>
GTAP_DEV uint32_t exchange(uint32_t x, bool low) {
  uint32_t a = x, b;
  if constexpr (D == 32 || D == 16) {
    // the row swaps of x with itself give both partners' keys to both lanes
    const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(x, x, false, false)
                           : __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = r[0];
    b = r[1];
  } else if constexpr (D == 8) {
    b = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x128, 0xF, 0xF, true));  // row_ror:8
  } else if constexpr (D == 4) {
    // half-row mirror (lane ^ 7), then the quad reversed (lane ^ 3)
    const int h = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x141, 0xF, 0xF, true);
    b = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, h, 0x1B, 0xF, 0xF, true));
  } else if constexpr (D == 2) {
    b = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x4E, 0xF, 0xF, true));
  } else {
    b = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xF, 0xF, true));
  }
  const uint32_t mn = a < b ? a : b, mx = a < b ? b : a;
  return low ? mn : mx;
}

// One merge round at lane distance D on N independent registers.
template <int D, uint32_t N>
GTAP_DEV void merge_round(uint32_t (&x)[N]) {
  const bool low = (lane_id() & static_cast<uint32_t>(D)) == 0;
#pragma unroll
  for (uint32_t i = 0; i < N; ++i) x[i] = exchange<D>(x[i], low);
}
// Ascending order of bitonic sequences over 2 D lanes each.
template <int D, uint32_t N>
GTAP_DEV void merge_from(uint32_t (&x)[N]) {
  merge_round<D>(x);
  if constexpr (D > 1) merge_from<D / 2>(x);
}

// One round of the sort's stage K (sorted runs of K lanes, alternating
// directions) at distance D.
template <int K, int D, uint32_t N>
GTAP_DEV void sort_round(uint32_t (&x)[N]) {
  const uint32_t ln = lane_id();
  const bool low = ((ln & static_cast<uint32_t>(D)) == 0) == ((ln & static_cast<uint32_t>(K)) == 0);
#pragma unroll
  for (uint32_t i = 0; i < N; ++i) x[i] = exchange<D>(x[i], low);
}
template <int K, int D, uint32_t N>
GTAP_DEV void sort_stage(uint32_t (&x)[N]) {
  sort_round<K, D>(x);
  if constexpr (D > 1) sort_stage<K, D / 2>(x);
}

// Sort each W keys of a register over their lanes, ascending.
template <int W, int K = 2, uint32_t N>
GTAP_DEV void sort_lanes(uint32_t (&x)[N]) {
  if constexpr (K < W) {
    sort_stage<K, K / 2>(x);
    sort_lanes<W, 2 * K>(x);
  } else {
    merge_from<W / 2>(x);
  }
}

// Ascending order of a bitonic sequence of 256 keys, key r * 64 + lane in x[r].
GTAP_DEV void merge_tile(uint32_t (&x)[kTileRegs]) {
#pragma unroll
  for (uint32_t r = 0; r < 2; ++r) {  // distance 128
    const uint32_t a = x[r], b = x[r + 2];
    x[r] = a < b ? a : b;
    x[r + 2] = a < b ? b : a;
  }
#pragma unroll
  for (uint32_t r = 0; r < 4; r += 2) {  // distance 64
    const uint32_t a = x[r], b = x[r + 1];
    x[r] = a < b ? a : b;
    x[r + 1] = a < b ? b : a;
  }
  merge_from<32>(x);
}

// A serial sort (nb unused) or merge as one lane described it; wave-uniform.
struct Span {
  const uint32_t *a, *b;
  uint32_t *out;
  uint32_t na, nb;
};

// Keys of a sorted range A followed by pads and the range B backwards: a
// bitonic sequence of 256 (na + nb <= 256).
GTAP_DEV void load_tile(const Span &s, uint32_t (&x)[kTileRegs]) {
#pragma unroll
  for (uint32_t r = 0; r < kTileRegs; ++r) {
    const uint32_t i = r * kWave + lane_id();
    const uint32_t j = kTile - 1 - i;
    x[r] = kPad;
    if (i < s.na) x[r] = co_ld32(s.a + i);
    else if (j < s.nb) x[r] = co_ld32(s.b + j);
  }
}
GTAP_DEV void store_tile(const Span &s, const uint32_t (&x)[kTileRegs]) {
#pragma unroll
  for (uint32_t r = 0; r < kTileRegs; ++r) {
    const uint32_t i = r * kWave + lane_id();
    if (i < s.na + s.nb) co_st32(s.out + i, x[r]);
  }
}

// Number of A's keys among the first d keys of merge(A, B), A's keys first on
// ties: A[i] is among them iff i < d and fewer than d - i of B's keys are
// smaller.  Each round all lanes test 64 equally spaced positions at once.
GTAP_DEV uint32_t merge_split(const Span &s, uint32_t d) {
  uint32_t lo = d > s.nb ? d - s.nb : 0u, hi = s.na < d ? s.na : d;  // the answer is in [lo, hi]
  while (lo < hi) {
    const uint32_t step = (hi - lo + kWave - 1) / kWave;
    const uint32_t i = lo + lane_id() * step;
    bool in = false;
    if (i < hi) in = co_ld32(s.b + (d - i - 1)) >= co_ld32(s.a + i);  // d - nb <= lo <= i < d
    const uint32_t c = static_cast<uint32_t>(__popcll(ballot(in)));
    const uint32_t base = lo;
    lo = c ? base + (c - 1) * step + 1 : base;
    const uint32_t top = base + c * step;
    hi = c && top > hi ? hi : top;
  }
  return lo;
}

GTAP_DEV uint64_t lane_u64(uint32_t lo, uint32_t hi, int k) {
  return static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lo), k))) |
         (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(hi), k))) << 32);
}

// A serial sort or merge as its lane describes it: addresses as two words.
struct Desc {
  uint32_t a[2], b[2], out[2], na, nb;
};

// Run the sorts (kMerge: merges) of the lanes in `m`, at most W keys each: the
// t-th takes W lanes, 4 * 64 / W of them at a time.  The descriptions move to
// the lanes [0, number of lanes in m) once.
template <int W, bool kMerge>
GTAP_DEV void run_short(uint64_t m, const Desc &d) {
  constexpr uint32_t N = 4, S = kWave / W;
  const uint32_t ln = lane_id(), count = static_cast<uint32_t>(__popcll(m)), i = ln % W;
  const int to = static_cast<int>(4 * ((m >> ln) & 1u ? rank_below(m) : count + rank_below(~m)));
  auto move = [&](uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_ds_permute(to, static_cast<int>(x)));
  };
  const Desc g{{move(d.a[0]), move(d.a[1])}, {kMerge ? move(d.b[0]) : 0u, kMerge ? move(d.b[1]) : 0u},
               {move(d.out[0]), move(d.out[1])}, move(d.na), kMerge ? move(d.nb) : 0u};
  for (uint32_t t0 = 0; t0 < count; t0 += N * S) {
    uint32_t *out[N];
    uint32_t len[N], x[N];
#pragma unroll
    for (uint32_t q = 0; q < N; ++q) {
      const uint32_t t = t0 + q * S + ln / W;
      auto of = [&](uint32_t v) {
        return static_cast<uint32_t>(__shfl(static_cast<int>(v), static_cast<int>(t % kWave), 64));
      };
      auto ptr = [&](const uint32_t (&w)[2]) {
        return reinterpret_cast<uint32_t *>(of(w[0]) | (static_cast<uint64_t>(of(w[1])) << 32));
      };
      const uint32_t *a = ptr(g.a), *b = kMerge ? ptr(g.b) : nullptr;
      const uint32_t na = of(g.na), nb = kMerge ? of(g.nb) : 0u;
      out[q] = ptr(g.out);
      len[q] = t < count ? na + nb : 0u;
      x[q] = kPad;
      if (t < count) {
        if (i < na) x[q] = co_ld32(a + i);
        else if (W - 1 - i < nb) x[q] = co_ld32(b + (W - 1 - i));
      }
    }
    if constexpr (kMerge) merge_from<W / 2>(x);
    else sort_lanes<W>(x);
#pragma unroll
    for (uint32_t q = 0; q < N; ++q)
      if (i < len[q]) co_st32(out[q] + i, x[q]);
  }
}

// The sorts or merges of the lanes in `m` that way, if all of them are short.
// (Widths of 16 for sorts and 32 for merges as well measured the same.)
GTAP_DEV bool run_short_sorts(uint64_t m, const Desc &d) {
  if ((ballot(d.na > 32) & m) != 0ull) return false;
  if ((ballot(d.na > 8) & m) == 0ull) run_short<8, false>(m, d);
  else run_short<32, false>(m, d);
  return true;
}
GTAP_DEV bool run_short_merges(uint64_t m, const Desc &d) {
  if ((ballot(d.na + d.nb > 64) & m) != 0ull) return false;
  if ((ballot(d.na + d.nb > 16) & m) == 0ull) run_short<16, true>(m, d);
  else run_short<64, true>(m, d);
  return true;
}

// Run the serial sorts of the lanes in `m` (span_of(k): lane k's).  Four at a
// time keep the DPP chains of one network apart and four loads in flight;
// the next four are loaded before the current ones are sorted.
template <class SpanFn>
GTAP_DEV void run_sorts(uint64_t m, SpanFn span_of) {
  constexpr uint32_t N = 4;
  Span cur[N], nxt[N];
  uint32_t x[N], y[N];
  uint64_t rest = m;
  auto load1 = [&](Span &s, uint32_t &v) {
    s.na = 0;
    v = kPad;
    if (rest) {
      s = span_of(__builtin_ctzll(rest));
      rest &= rest - 1;
      if (lane_id() < s.na) v = co_ld32(s.a + lane_id());
    }
  };
  auto load = [&](Span (&s)[N], uint32_t (&v)[N]) {
    load1(s[0], v[0]);
    load1(s[1], v[1]);
    load1(s[2], v[2]);
    load1(s[3], v[3]);
  };
  load(cur, x);
  for (;;) {
    const bool more = rest != 0;
    if (more) load(nxt, y);
    sort_lanes<64>(x);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i)
      if (lane_id() < cur[i].na) co_st32(cur[i].out + lane_id(), x[i]);
    if (!more) break;
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) {
      cur[i] = nxt[i];
      x[i] = y[i];
    }
  }
}

// Run the serial merges of the lanes in `m`.  A merge longer than a tile is
// cut into tiles of 256 outputs at the split points of its merge path.
template <class SpanFn>
GTAP_DEV void run_merges(uint64_t m, SpanFn span_of) {
  uint64_t rest = m;
  Span whole{nullptr, nullptr, nullptr, 0, 0};  // what is left of the current merge
  // the next tile, or an empty one at the end
  auto next = [&]() -> Span {
    while (whole.na + whole.nb == 0) {
      if (rest == 0) return whole;
      whole = span_of(__builtin_ctzll(rest));
      rest &= rest - 1;
    }
    Span t = whole;
    if (whole.na + whole.nb > kTile) {
      t.na = merge_split(whole, kTile);
      t.nb = kTile - t.na;
    }
    whole.a += t.na;
    whole.b += t.nb;
    whole.na -= t.na;
    whole.nb -= t.nb;
    whole.out += t.na + t.nb;
    return t;
  };
  constexpr uint32_t N = 2;
  Span cur[N], nxt[N];
  uint32_t x[N][kTileRegs], y[N][kTileRegs];
  auto load = [&](Span (&s)[N], uint32_t (&v)[N][kTileRegs]) {
    s[0] = next();
    load_tile(s[0], v[0]);
    s[1] = next();
    load_tile(s[1], v[1]);
  };
  load(cur, x);
  while (cur[0].na + cur[0].nb != 0) {
    load(nxt, y);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) merge_tile(x[i]);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) store_tile(cur[i], x[i]);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) {
      cur[i] = nxt[i];
#pragma unroll
      for (uint32_t r = 0; r < kTileRegs; ++r) x[i][r] = y[i][r];
    }
  }
}

}  // namespace cilk
}  // namespace gtap
