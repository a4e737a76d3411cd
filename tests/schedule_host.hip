// The tile schedule's arithmetic on the host: what a launch's workgroups work
// out, with plain loops in place of the wave's scans and searches.
#include <algorithm>
#include <vector>

#include "schedule.h"

using namespace sched;

extern "C" int host_counts_tiles(int g, int Hkv, int C_max, int B, int tiles) {
  return counts_tiles(Launch{g, Hkv, C_max, 0, 0}, B, tiles);
}

// seqs[B]: packed lengths.  head: Pe, whole, Wt, width, longer.  Per range, 11
// words: g0, g1, first tile's b, kvh and j, last unit's b and kvh, and the first
// and last owner of the first tile's unit and of the last one's.
extern "C" void host_schedule(int g, int Hkv, int C_max, int P, int flat, int tile_keys, int B, const uint32_t* seqs,
                              int64_t* head, int32_t* ranges) {
  const Launch p = {g, Hkv, C_max, P, flat};
  std::vector<int> pref(B + 1), cpref(B + 1);
  int with_tiles = 0;
  for (int b = 0; b < B; ++b) {
    const int n = seq_tiles(seqs[b], tile_keys);
    pref[b + 1] = pref[b] + n;
    with_tiles += n > 0;
  }
  Sched sc;
  sc.whole = 0;
  const int N = pref[B] * Hkv;
  if (B <= 64 && !flat)
    sc.whole = pick_whole(
        p, N, with_tiles * Hkv,
        [&](int t) {
          int k = 0;
          for (int b = 0; b < B; ++b) k += (seq_tiles(seqs[b], tile_keys) + t - 1) / t;
          return k;
        },
        [&](int t) {
          int e = 0;
          for (int b = 0; b < B; ++b) e = std::max(e, range_excess(p, seq_tiles(seqs[b], tile_keys), seqs[b], t));
          return e;
        },
        [&]() {
          int c = 0;
          for (int b = 0; b < B; ++b) c += unit_cost(p, seq_tiles(seqs[b], tile_keys), seqs[b], 0);
          return c;
        });
  for (int b = 0; b < B; ++b)
    cpref[b + 1] = cpref[b] + unit_cost(p, seq_tiles(seqs[b], tile_keys), seqs[b], sc.whole);
  sc.cut(p, N, cpref[B]);
  head[0] = sc.Pe;
  head[1] = sc.whole;
  head[2] = sc.Wt;
  head[3] = sc.width;
  head[4] = sc.longer;
  auto seq_at = [&](uint32_t X) {
    At a;
    a.b = 0;
    for (int b = 0; b < B; ++b)
      if ((uint32_t)cpref[b] * (uint32_t)Hkv <= X) a.b = b;
    a.s = seqs[a.b];
    a.n = seq_tiles(a.s, tile_keys);
    a.t0 = pref[a.b] * Hkv;
    a.c0 = (uint32_t)cpref[a.b] * (uint32_t)Hkv;
    a.U = (uint32_t)unit_cost(p, a.n, a.s, sc.whole);
    return a;
  };
  for (int q = 0; q < sc.Pe; ++q) {
    const Range r = range_of(p, sc, q, seq_at);
    const int32_t row[11] = {r.g0, r.g1, r.first.b, r.kvh, r.j, r.last.b, r.kvl,
                             sc.owner(r.cf), sc.last_owner(p, r.first.s, r.first.n, r.cf),
                             sc.owner(r.cl), sc.last_owner(p, r.last.s, r.last.n, r.cl)};
    for (int i = 0; i < 11; ++i) ranges[11 * q + i] = row[i];
  }
}
