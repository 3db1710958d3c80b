// plan.h -- host-side rules of the dot calls that need no GPU: who may use a
// context's scratch, how a K loop is split, and which kernel takes what of a
// rotation call.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace imc {

// Which stream may use a context's parts scratch: the first whose call splits a
// K loop, for the life of the context, since only one stream's calls are known
// to run in order.  Not lent to captured calls (a graph may be replayed beside
// eager calls) nor to the per-thread default stream, whose one handle names
// another stream in every thread.
struct PartsOwner {
  std::atomic<bool> owned{false};
  std::atomic<uintptr_t> stream{0};   // valid once owned
  bool lends(uintptr_t to, bool per_thread, bool capturing) const {
    return !capturing && !per_thread && (!owned || stream == to);
  }
  void take(uintptr_t by) {   // one caller at a time
    stream = by;
    owned = true;
  }
};

// Workgroups that share one tile's K loop: as many as find a CU (`per_cu`
// workgroups each, of `cus`) beside the call's `tiles`, at most `units` of the
// loop's pieces and what `bytes` of scratch hold (`outputs` u32 a part).  1: no
// split.
inline uint32_t dot_splits(uint64_t tiles, uint32_t per_cu, uint32_t units, uint64_t outputs, size_t bytes, int cus) {
  if (bytes == 0 || cus <= 0 || tiles == 0 || outputs == 0) return 1;
  uint64_t s = uint64_t(cus) * per_cu / tiles;
  s = s < units ? s : units;
  const uint64_t fit = bytes / 4 / outputs;
  s = s < fit ? s : fit;
  return s < 1 ? 1 : uint32_t(s);
}

// Row tiles of `m` rows.
inline uint64_t rot_tiles(uint64_t rows, uint64_t m) { return (rows + m - 1) / m; }

// Whether every one of `mt` row tiles' workgroups finds a CU at once, of `nt`
// column tiles over `vecs` vectors: a column tile's workgroups run on one of the
// 8 XCDs.
inline bool one_round(uint64_t mt, uint64_t nt, uint32_t vecs, int cus) {
  return cus >= 8 && mt * ((nt + 7) / 8) * vecs <= uint64_t(cus) / 8;
}

// Rows of a tile (64 .. 256) of a rotation call whose loop is not split: the
// fewest that still leave a CU for every tile.  Such a call takes as long as one
// tile, and a tile of 64 rows takes half of a whole one's time.
inline uint32_t rot_tile_rows(uint64_t rows, uint64_t nt, uint32_t vecs, int cus) {
  for (uint32_t m = 64; m < 256; m += 64)
    if (one_round(rot_tiles(rows, m), nt, vecs, cus)) return m;
  return 256;
}

// What a call may use: scratch for the parts of its loops, CUs, and the angular
// segments of its K loop.
struct DotRoom {
  size_t bytes;
  int cus;
  uint32_t segs;
};
constexpr uint32_t rot_segs(bool galois) { return galois ? 16 : 32; }

// Workgroups that share one tile's segments in a rotation call, one per CU (its
// LDS).  The launch rounds a workgroup's segments up.
inline uint32_t rot_splits(uint64_t rows, uint64_t n, uint32_t vecs, const DotRoom& room) {
  const uint64_t tiles = rot_tiles(rows, 256) * ((n + 127) / 128) * vecs;
  return dot_splits(tiles, 1, room.segs, rows * n * vecs, room.bytes, room.cus);
}

// Row tiles of a launch that go first: all but a last one of up to 128 rows,
// whose workgroups are the shorter ones, so that they fill the ends of the CUs'
// work; in the column tiles' order they would keep the longer tiles of a
// column apart.  A launch of many rounds has no ends to fill and reads the
// database once less in one order.  us, in order / apart, 65,536 entries, 15
// rotations: 18 queries 3,599 / 3,214, 40 5,676 / 5,397, 52 7,247 / 6,920, 70
// (20 rounds of one tile per CU) 8,987 / 8,798; last tiles of 163 and 192
// rows no better (5,979 / 6,004, 7,706 / 7,948); 40 queries against 300,000
// (55 rounds) 24,718 / 24,911, 64 x 17 against 100,000 (31) 13,733 / 13,981.
inline uint32_t rot_lead_tiles(uint64_t rows, uint64_t tiles, int cus) {
  const uint32_t mt = uint32_t(rot_tiles(rows, 256));
  return mt > 1 && rows - uint64_t(mt - 1) * 256 <= 128 && tiles <= 24 * uint64_t(cus) ? mt - 1 : mt;
}

// ---------------------------------------------------------------------------
// Which kernel takes what of a call at r >= 13 rotations.  Times are counted
// in units of 5 us of the replicated form.  A call takes its tiles in rounds
// of one per CU; a tile's time, from 65,536 entries (ms / rounds): rot_dot.hip
// 2 queries 1.14 / 4, 4: 1.42 / 4, 6: 1.75 / 4, 8: 2.11 / 4 (one row tile), 16:
// 3.90 / 8, 32: 7.45 / 16, 64: 14.5 / 32; pairs 8 queries 2.65 / 4, 10: 3.06 /
// 4, 12: 3.06 / 4, 16: 3.39 / 4 (one query tile), 32: 5.86 / 8, 64: 10.9 / 16.
// The last round is rarely full, and up to 8 queries past a multiple of 16
// leave half of a pairs' tile idle: those columns and those queries may go to
// rot_dot.hip's kernel in calls of their own, which splits its loop when its
// tiles are few.  us, one launch / as planned: 16 queries x 20,011 entries
// 1,370 / 1,097, 18 x 65,536 5,420 / 4,490, 7 queries x 15 rotations x 20,000
// 585 / 480.
// ---------------------------------------------------------------------------
constexpr uint64_t kLaunchCost = 2;
constexpr uint32_t kRotCols = 128, kPairQueries = 16;   // entries of a column tile, queries of a pairs' tile

// A rot_dot.hip tile alone in its columns, and beside others.
inline uint64_t rot_tile_cost(uint64_t rows) { return rows <= 64 ? 56 : rows <= 128 ? 68 : rows <= 192 ? 86 : 105; }
constexpr uint64_t kRotSharedCost = 94;
inline uint64_t pair_tile_cost(uint64_t q) { return q > 16 ? 142 : q > 12 ? 168 : q > 8 ? 153 : 132; }

// More parts than these, in replicated calls of up to 8 tiles, save up to 3 of
// a call's units, which is less than the model is true to: counted, they change
// the route of 4 in 200,000 random calls, to 1.03, 1.04, 0.64 and 0.66 of the
// speed.
constexpr uint32_t kPlanSplits = 16;

// The shorter tiles of few that all run at once are not counted here: the model
// would take the last round of calls that don't split apart, which then waits for
// the rounds before it (us, whole / apart: 56 queries of 26 rotations x 46,052
// entries 3,978 / 4,351, 44 of 15 x 23,261 Galois 618 / 664, 13 of 31 x 17,337 578 /
// 627).
inline uint64_t rot_cost(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (q == 0 || n == 0) return 0;
  const uint64_t rows = q * r, mt = rot_tiles(rows, 256), cols = (n + kRotCols - 1) / kRotCols * vecs;
  const uint32_t splits = rot_splits(rows, n, vecs, room);
  if (splits > 1) return 2 * kLaunchCost + rot_tile_cost(rows) / (splits < kPlanSplits ? splits : kPlanSplits) + 2;
  const auto rounds = [&](uint64_t tiles) { return (tiles + room.cus - 1) / room.cus; };
  const uint64_t lead = rot_lead_tiles(rows, mt * cols, room.cus);
  return kLaunchCost + (lead > 1 ? kRotSharedCost : rot_tile_cost(rows)) * rounds(lead * cols) +
         (lead < mt ? rot_tile_cost(rows - lead * 256) * rounds(cols) : 0);
}

// Column tiles that fill whole rounds, `per` tiles each.
inline uint64_t full_cols(uint64_t n, uint64_t per, const DotRoom& room) {
  return (n + kRotCols - 1) / kRotCols * per / room.cus * room.cus / per;
}

// rot_dot.hip's columns that go in a first call, the whole rounds; all n of
// them if the last round is better not taken apart.
inline uint64_t rot_first_cols(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (room.cus <= 0) return n;
  const uint64_t m = full_cols(n, rot_tiles(q * r, 256) * vecs, room) * kRotCols;
  if (m == 0 || m >= n) return n;
  return rot_cost(q, r, m, vecs, room) + rot_cost(q, r, n - m, vecs, room) < rot_cost(q, r, n, vecs, room)
             ? m
             : n;
}

inline uint64_t rot_rounds_cost(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (q == 0 || n == 0) return 0;
  const uint64_t m = rot_first_cols(q, r, n, vecs, room);
  return rot_cost(q, r, m, vecs, room) + rot_cost(q, r, n - m, vecs, room);
}

// A call that runs whole in shorter tiles, all at once; none if that is not so.
inline uint64_t rot_short_cost(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  const uint32_t m = rot_tile_rows(q * r, (n + kRotCols - 1) / kRotCols, vecs, room.cus);
  return m < 256 && rot_splits(q * r, n, vecs, room) == 1 ? kLaunchCost + rot_tile_cost(m) : UINT64_MAX;
}

struct RotPlan {
  uint32_t q;   // queries and columns of the pairs; the rest is rot_dot.hip's
  uint64_t n;
};

// Pairs take lists of 27 .. 31 consecutive rotations, ascending.
inline RotPlan rot_plan(uint32_t q_all, uint32_t r, const int8_t* rot, uint64_t n_all, uint32_t vecs,
                        const DotRoom& room) {
  const RotPlan none{0, 0};
  if (r < 27 || r > 31 || room.cus <= 0) return none;
  for (uint32_t i = 1; i < r; ++i)
    if (rot[i] != rot[0] + int(i)) return none;
  RotPlan best = none;
  // us, pairs / shorter tiles: 9 queries of 30 rotations x 632 entries Galois 264 /
  // 103, 28 of 30 x 1,405 507 / 196
  uint64_t least = rot_rounds_cost(q_all, r, n_all, vecs, room);
  const uint64_t in_short_tiles = rot_short_cost(q_all, r, n_all, vecs, room);
  least = in_short_tiles < least ? in_short_tiles : least;
  const uint32_t over = q_all % kPairQueries;
  for (int less = 0; less < 2; ++less) {
    if (less && (over == 0 || over > kPairQueries / 2)) break;
    const uint32_t q = less ? q_all - over : q_all;
    if (q == 0) break;
    const uint64_t per = uint64_t(q + kPairQueries - 1) / kPairQueries * vecs, nt = (n_all + kRotCols - 1) / kRotCols;
    const uint64_t full = full_cols(n_all, per, room);
    for (int part = 0; part < 2; ++part) {
      const uint64_t cols = part ? full : nt;
      if (cols == 0 || (part && cols == nt)) break;
      const uint64_t n = cols * kRotCols < n_all ? cols * kRotCols : n_all;
      const uint64_t cost = kLaunchCost + pair_tile_cost(q) * ((cols * per + room.cus - 1) / room.cus) +
                            rot_rounds_cost(q, r, n_all - n, vecs, room) +
                            rot_rounds_cost(q_all - q, r, n_all, vecs, room);
      if (cost < least) {
        least = cost;
        best = RotPlan{q, n};
      }
    }
  }
  return best;
}

}  // namespace imc
