// Tile schedule of the verification attention kernel: which tiles of a launch
// each workgroup takes.  Plain 32-bit arithmetic on the lengths and their
// prefix sums, the same in the kernel and, compiled for the host, in its CPU
// test; the kernel supplies the sums and searches over the sequences.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sched {

#define SCHED_FN __host__ __device__ __forceinline__

constexpr int kBlk = 16;   // keys (and query rows) per MFMA block

// Launch constants
struct Launch {
  int g, Hkv, C_max;   // query heads per KV head, KV heads, most chunk tokens of a sequence
  int P;               // workgroups
  int flat;            // the schedule counts tiles, not their costs (totals past 32 bits)
};

// Lengths of a sequence, packed as (T << 8) | c: context and chunk, chunk
SCHED_FN int seq_T(uint32_t s) { return (int)(s >> 8); }
SCHED_FN int seq_c(uint32_t s) { return (int)(s & 0xffu); }
// key tiles of each of its units
SCHED_FN int seq_tiles(uint32_t s, int tile_keys) {
  return seq_c(s) == 0 ? 0 : (seq_T(s) + tile_keys - 1) / tile_keys;
}

// Cost of one tile of a sequence with c chunk tokens: a fixed part for
// streaming the tile, plus one per 16-row block of the unit's c * g query
// rows.  A unit with many rows can take longer on a tile than the tile's
// HBM stream lasts, so workgroups get equal cost rather than equal tiles.
// The weights follow measured tile times (ragged chunks, 1-7 row blocks:
// 2.7, 3.1 and 3.3 us per tile for 1-2, 3-4 and 5-7 blocks).
constexpr int kTileCost = 10;
SCHED_FN int tile_cost(const Launch& p, uint32_t s, int whole) {
  return whole || p.flat ? 1 : kTileCost + (seq_c(s) * p.g + kBlk - 1) / kBlk;
}
// Extra costs of a unit: at its start (a first tile that is mostly partial,
// the switch of Q) and at its end (the result's stores and, for units of one
// or two row blocks, the merge of the key-split states; charged after its
// last tile), so ranges that cross more unit boundaries get fewer tiles.  A
// range that starts inside a unit pays for that unit's end.  (Measured: on
// B = 64 with chunks of 5 and 4 query heads per KV head a unit end holds a
// workgroup ~1.6 us and its start ~0.6 us, against ~2.2 us per tile; a fit
// over eight splits of the tree workload, four row blocks per unit, gives
// 2.2 us per unit and 2.3 per tile: with 3 + 6 for it, not 6 + 0, 77.9 -> 77.0
// us per call, ragged chunks 123.1 -> 122.5.)
constexpr int kStartSplit = 3, kEndSplit = 9;   // units of one or two row blocks
constexpr int kStartRest = 3, kEndRest = 6;     // larger units
constexpr int kExtraMax =
    kStartSplit + kEndSplit > kStartRest + kEndRest ? kStartSplit + kEndSplit : kStartRest + kEndRest;
SCHED_FN bool split_unit(const Launch& p, uint32_t s) { return seq_c(s) * p.g <= 2 * kBlk; }
SCHED_FN int start_cost(const Launch& p, uint32_t s, int whole) {
  return whole || p.flat ? 0 : split_unit(p, s) ? kStartSplit : kStartRest;
}
SCHED_FN int end_cost(const Launch& p, uint32_t s) {
  return p.flat ? 0 : split_unit(p, s) ? kEndSplit : kEndRest;
}
// the most that a tile costs with its unit's start and end
SCHED_FN int most_cost(const Launch& p) {
  return p.flat ? 1 : kTileCost + (p.C_max * p.g + kBlk - 1) / kBlk + kExtraMax;
}
// A launch of B sequences of at most `tiles` tiles per unit counts tiles if
// their costs could add up to 2^31.
SCHED_FN int counts_tiles(const Launch& p, int B, int tiles) {
  const int64_t unit = (int64_t)tiles * (kTileCost + (p.C_max * p.g + kBlk - 1) / kBlk) + kExtraMax;
  return (int64_t)B * p.Hkv * unit >= ((int64_t)1 << 31);
}
// cost of one unit (one KV head) of a sequence with packed lengths s: its n
// tiles, its start and its end; with `whole`, its tiles rounded up to whole
// ranges
SCHED_FN int unit_cost(const Launch& p, int n, uint32_t s, int whole) {
  if (whole) return (n + whole - 1) / whole * whole;
  return n > 0 ? n * tile_cost(p, s, 0) + start_cost(p, s, 0) + end_cost(p, s) : 0;
}

// Launches of few units (at most half the workgroups, one sequence per lane of
// the scheduling wave): ranges are cut inside units only, `whole` tiles each,
// so that no workgroup ends two units or holds two pieces: a second unit in a
// range costs its end (1.2 us), and often the publication and merge of a
// second piece, as much as one or two tiles of a launch that has two to
// twenty per workgroup.  `whole` is the smallest that leaves at most one range
// per workgroup, of kWholeTries from the even share on (past those the uneven
// last ranges of units waste more), but at least kWholeMin (ranges of one tile
// pay more for their merge than they save), and kWholeUnit where that makes
// units whole on average.  Against equal cost: 8 KV heads, B = 1 with 300
// tokens 12.4 -> 10.5 us, B = 8 with 512-2048 21.9 -> 19.4, B = 16 with 300-900
// 20.8 -> 18.2, B = 2 with 16k 33.7 -> 31.0, B = 4 with 20-30k 72.3 -> 71.2;
// B = 4 with 512-2048 (two tiles per range either way) 15.5 -> 15.6.
//
// Ranges of a fixed number of tiles are uneven where units differ in rows or
// leave short last ranges, and the launch ends with the longest.  Where that
// one costs over kWholeUneven half tiles more than the average range (a
// quarter of it taken over all workgroups, idle ones too), cost is cut equally
// after all: 4 KV heads of 7 query heads, chunks of 1-16, B = 28 with 1-10k
// tokens 74.9 us in ranges of 21 tiles, 67.8 at equal cost; B = 24 with 3800,
// 192 ranges of 15 tiles, 56.9 and 54.2; 2 KV heads, fp32, B = 56 with
// 128-3000 53.7 and 48.5.  Even ranges on fewer workgroups stream as fast: 8
// KV heads, B = 12 with 3800 tokens, 192 ranges of 15 tiles, 39.1 us, at equal
// cost 41.0.  Over 500 launches timed both ways, the form chosen takes 0.5%
// longer than the better one of each with 6 to 8 half tiles, 0.8% with 4 and
// 0.8% without a limit.  Not asked of ranges of up to kWholeShort tiles: such
// launches would notice the two reductions (0.1 us), and none of the 500 is
// uneven enough.
//
// N tiles and `units` units in all.  ranges(t): ranges of t tiles per KV head;
// excess(t): the most, over the sequences, of range_excess; cost(): of one KV
// head's units.
constexpr int kWholeUnit = 3, kWholeMin = 2, kWholeTries = 4, kWholeUneven = 7, kWholeShort = 4;
// twice the cost of a sequence's longest range of t tiles, less kWholeUneven of
// its half tiles
SCHED_FN int range_excess(const Launch& p, int n, uint32_t s, int t) {
  if (n == 0) return 0;
  return (2 * (n < t ? n : t) - kWholeUneven) * tile_cost(p, s, 0) + 2 * (start_cost(p, s, 0) + end_cost(p, s));
}
template <class RANGES, class EXCESS, class COST>
SCHED_FN int pick_whole(const Launch& p, int N, int units, RANGES ranges, EXCESS excess, COST cost) {
  if (units == 0 || 2 * units > p.P) return 0;
  int t = N <= kWholeUnit * units ? kWholeUnit : kWholeMin;
  if (N > t * p.P) t = (N + p.P - 1) / p.P;
  for (int tries = 0; tries < kWholeTries; ++tries, ++t) {
    const int k = ranges(t);
    if (k * p.Hkv <= p.P) {
      if (__builtin_expect(t > kWholeShort, 0) && 2 * (int64_t)excess(t) * k * p.P > (int64_t)cost() * (3 * p.P + k * p.Hkv))
        return 0;
      return t;
    }
  }
  return 0;
}

// Tile schedule shared by every workgroup of a launch.  The tiles of all
// units form one list [0, N) in (sequence, KV head, tile) order; tile j of
// unit kvh of sequence b starts at cost Hkv cpref[b] + kvh U_b + (j > 0 ?
// S_b + j w_b : 0), cpref[b] the cost of one KV head's units of the sequences
// before b, w_b its sequence's tile cost, S_b and E_b its unit-start and
// unit-end costs and U_b = n_b w_b + S_b + E_b a unit's cost, out of Wt
// in all.  The costs [0, Wt) are cut into Pe ranges, the first Wt mod Pe of
// them one longer than the rest (width); range q holds the tiles whose start
// cost lies in it.  With Pe <= Wt / max_b (w_b + S_b + E_b) no range is
// empty, since consecutive tile starts are at most max_b (w_b + S_b + E_b)
// apart.  Everything fits 32 bits: a launch whose total cost could reach 2^31
// counts tiles instead (Launch::flat), fewer than 2^30 (host check).  The
// search sits ahead of every workgroup's first load, and the list of shared
// units ahead of its first tile's compute: with 64-bit costs and
// double-precision quotients the first took 1.5 us and a call on two
// sequences began to compute 6.0 us into the launch; in 32 bits 0.8 us and
// 4.0 us (B = 4, 24 MB of K and V: 19.3 -> 17.5 us per call; B = 64, 347 MB:
// 63.8 -> 63.2 us, as the stream makes up for most of it).
struct Sched {
  int Pe, whole;
  uint32_t Wt, width, longer;
  // N tiles in all, cost_per_head the cost of one KV head's units
  SCHED_FN void cut(const Launch& p, int N, int cost_per_head) {
    Wt = (uint32_t)p.Hkv * (uint32_t)cost_per_head;
    const uint32_t most = (uint32_t)most_cost(p);
    if (whole) {
      Pe = (int)(Wt / (uint32_t)whole);
    } else if (Wt >= (uint32_t)p.P * most) {
      Pe = p.P;
    } else {   // at least one range when there are tiles
      const int fit = (int)(Wt / most);
      Pe = N == 0 ? 0 : fit < 1 ? 1 : fit;
    }
    width = Wt / (uint32_t)(Pe > 1 ? Pe : 1);
    longer = Wt - width * (uint32_t)Pe;
  }
  SCHED_FN uint32_t bound(int q) const {   // range q's first cost
    return (uint32_t)q * width + ((uint32_t)q < longer ? (uint32_t)q : longer);
  }
  // range of the tile that starts at cost c
  SCHED_FN int owner(uint32_t c) const {
    const uint32_t cut = longer * (width + 1);
    const bool low = c < cut;
    return (int)((low ? c : c - cut) / (low ? width + 1 : width) + (low ? 0 : longer));
  }
  // ranges of the first and the last of the n tiles of a unit that starts at
  // cost c
  SCHED_FN int last_owner(const Launch& p, uint32_t s, int n, uint32_t c) const {
    return owner(n > 1 ? c + (uint32_t)(start_cost(p, s, whole) + (n - 1) * tile_cost(p, s, whole)) : c);
  }
};

// The sequence whose units hold a cost, and the tiles and the cost before them
struct At {
  int b, n, t0;   // sequence, tiles per unit, tiles before its units
  uint32_t s, c0, U;   // packed lengths, cost before its units, cost of a unit
};

// Tiles [g0, g1) of a range, with the sequence, KV head and index of the first
// one, the sequence and KV head of the last one, and the costs at which the
// units of both start
struct Range {
  int g0, g1, kvh, j, kvl;
  At first, last;
  uint32_t cf, cl;
};

// Range q < Pe.  seq_at(X): the last sequence b with Hkv cpref[b] <= X < Wt (it
// has tiles, as the next prefix is past X).
template <class SEQ_AT>
SCHED_FN Range range_of(const Launch& p, const Sched& sc, int q, SEQ_AT seq_at) {
  Range r;
  // the first tile that starts at or after the range's first cost, ...
  const uint32_t X = sc.bound(q);
  At f = seq_at(X);
  uint32_t kvh = (X - f.c0) / f.U;
  uint32_t cf = f.c0 + kvh * f.U;
  const uint32_t w = (uint32_t)tile_cost(p, f.s, sc.whole), S = (uint32_t)start_cost(p, f.s, sc.whole), x = X - cf;
  uint32_t j = x == 0 ? 0 : x <= S ? 1 : (x - S + w - 1) / w;
  // (rounded up to a unit's end: the next unit's first tile)
  r.g0 = f.t0 + (int)kvh * f.n + ((int)j < f.n ? (int)j : f.n);
  if ((int)j >= f.n) {
    j = 0;
    cf += f.U;
    if ((int)++kvh == p.Hkv) {
      kvh = 0;
      f = seq_at(cf);
    }
  }
  // ... and the last one that starts before its end
  const uint32_t Y = sc.bound(q + 1) - 1;
  const At e = seq_at(Y);
  const uint32_t kvl = (Y - e.c0) / e.U;
  const uint32_t cl = e.c0 + kvl * e.U;
  const uint32_t wl = (uint32_t)tile_cost(p, e.s, sc.whole), Sl = (uint32_t)start_cost(p, e.s, sc.whole), y = Y - cl;
  const int i = y < Sl + wl ? 0 : (int)((y - Sl) / wl);
  r.g1 = e.t0 + (int)kvl * e.n + (i < e.n - 1 ? i : e.n - 1) + 1;
  r.kvh = (int)kvh;
  r.j = (int)j;
  r.kvl = (int)kvl;
  r.first = f;
  r.last = e;
  r.cf = cf;
  r.cl = cl;
  return r;
}

}  // namespace sched
