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
// LDS), and no more than run at once on the XCDs of their columns: two rounds of
// half a loop are no faster than a whole one (31 rotations, code and mask, us: 48
// queries x 1,280 entries in 2 parts 430, whole in 192-row tiles 330; 24 x 1,792 in 3
// parts 292, in 2 214; 80 x 512 in 4 parts 301, in 3 213).  The launch rounds a
// workgroup's segments up.
inline uint32_t rot_splits(uint64_t rows, uint64_t n, uint32_t vecs, const DotRoom& room) {
  const uint64_t mt = rot_tiles(rows, 256), nt = (n + 127) / 128;
  uint32_t s = dot_splits(mt * nt * vecs, 1, room.segs, rows * n * vecs, room.bytes, room.cus);
  while (s > 1 && room.cus >= 8 && !one_round(mt, nt * s, vecs, room.cus)) --s;
  return s;
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
// Which kernel takes what of a call at r >= 13 rotations.  Times in us of the
// replicated form (Galois-ring shares take half of each alike).
//
// A column tile's workgroups run on one XCD, one to a CU, so a launch runs in
// rounds of the XCD that has the most column tiles.  A full round takes longer
// than a sparse one (the part is power-bound: few busy CUs run at a higher clock);
// up to half of the CUs take no longer than one.  Measured, 31 rotations, one
// launch, the code dot alone (us; column tiles):
//   rot_dot.hip   1 query 140 (8) 156 (64) 172 (128) 275 (256) 546 (512), 8 194 (8)
//     224 (64) 318 (128) 408 (140) 529 (256) 1,061 (512), 16 194 (8) 302 (64) 489 (128)
//     825 (140) 979 (256), 64 201 (8) 438 (32) 806 (40) 923 (64) 1,242 (72) 1,844 (128);
//   pair_dot.hip  8 queries 339 (8) 460 (128) 533 (192), 16 506 (8) 572 (128) 705 (192),
//     32 507 (8) 554 (64) 739 (128) 1,197 (140), 64 508 (8) 698 (64) 1,157 (72) 1,409 (128).
// The costs below give 1,667 such launches within -8 and +15 % in nine of ten.
//
// The last round is rarely full, and up to 8 queries past a multiple of 16 leave
// half of a pairs' tile idle: those columns and those queries may go to
// rot_dot.hip's kernel in calls of their own, which splits its loop when its tiles
// are few.  Columns are taken apart by eights, one for each XCD: 18 of 25 in the
// first call (80 queries of 22 rotations x 3,133 entries, all CUs counted as one)
// are two rounds on two of the XCDs, 1,010 us against 825 in one launch.
// ---------------------------------------------------------------------------
constexpr uint32_t kRotCols = 128, kPairQueries = 16;   // entries of a column tile, queries of a pairs' tile
constexpr uint64_t kLaunchCost = 5;

struct TileCost {
  uint64_t sparse, full;   // a round of few tiles, one of a tile on every CU
};
// A rot_dot.hip tile of this many rows, alone in its columns.
inline TileCost rot_tile_cost(uint64_t rows) {
  return rows <= 32    ? TileCost{140, 275}
         : rows <= 64  ? TileCost{190, 290}
         : rows <= 128 ? TileCost{200, 360}
         : rows <= 192 ? TileCost{235, 440}
                       : TileCost{310, 530};
}
// One beside others of its columns.
inline TileCost rot_shared_cost(uint32_t m) {
  return m == 64 ? TileCost{192, 230} : m == 128 ? TileCost{250, 310} : m == 192 ? TileCost{300, 385} : TileCost{310, 475};
}
inline TileCost pair_tile_cost(uint64_t q) {
  return q <= 8 ? TileCost{400, 635} : q <= 12 ? TileCost{490, 765} : q <= 16 ? TileCost{505, 825}
       : q <= 32 ? TileCost{505, 735} : TileCost{505, 710};
}

// Column tiles of the XCD that has the most.
inline uint64_t xcd_cols(uint64_t cols) { return (cols + 7) / 8; }

// `tiles` workgroups on an XCD.
inline uint64_t rounds_cost(uint64_t tiles, TileCost c, int cus) {
  const uint64_t cx = uint64_t(cus) / 8, before = (tiles - 1) / cx, last = tiles - before * cx;
  return before * c.full + c.sparse + (2 * last > cx ? (c.full - c.sparse) * (2 * last - cx) / cx : 0);
}

// A whole loop in tiles of m rows, `cols` column tiles over all vectors on an XCD.
inline uint64_t rot_loop_cost(uint64_t rows, uint32_t m, uint64_t cols, int cus) {
  const uint64_t mt = rot_tiles(rows, m), last = rows - (mt - 1) * m;
  if (mt == 1) return rounds_cost(cols, rot_tile_cost(last), cus);
  TileCost c = rot_shared_cost(m);
  if (m < 256) return rounds_cost(cols * mt, c, cus);
  const TileCost short_one = rot_tile_cost(last);
  const uint64_t alone = rot_tile_cost(256).full, cx = uint64_t(cus) / 8;
  if (last > 128 || cols * mt <= cx) {
    const uint64_t equal = (cols * (mt - 1) * alone + cols * short_one.full + alone - 1) / alone;
    return rounds_cost(equal > cx || cols * mt <= cx ? equal : cols * mt, c, cus);
  }
  // short last tiles after the others, and beside their last round
  if (mt == 2) c.full = alone;
  const uint64_t beside = (cx - cols * (mt - 1) % cx) % cx;
  return rounds_cost(cols * (mt - 1), c, cus) + (cols > beside ? rounds_cost(cols - beside, short_one, cus) : 0);
}

// One call of rot_dot.hip's kernel.
inline uint64_t rot_cost(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (q == 0 || n == 0) return 0;
  const uint64_t rows = q * r, nt = (n + kRotCols - 1) / kRotCols;
  const uint32_t splits = rot_splits(rows, n, vecs, room);
  if (splits > 1) {
    const uint32_t per = (room.segs + splits - 1) / splits, parts = (room.segs + per - 1) / per;
    return 3 * kLaunchCost + rot_loop_cost(rows, 256, xcd_cols(nt * parts) * vecs, room.cus) * per / room.segs;
  }
  return kLaunchCost + rot_loop_cost(rows, rot_tile_rows(rows, nt, vecs, room.cus), xcd_cols(nt) * vecs, room.cus);
}

// Column tiles whose `per` workgroups each fill whole rounds of every XCD.
inline uint64_t full_cols(uint64_t n, uint64_t per, const DotRoom& room) {
  const uint64_t cx = uint64_t(room.cus) / 8, nt = (n + kRotCols - 1) / kRotCols;
  return xcd_cols(nt) * per / cx * cx / per * 8;
}

// A call is taken apart when the model gives it 1/24 of the time or 50 us, a tenth of
// a round: whole rounds cost the same either way, and less is within its error.
inline bool clearly_less(uint64_t cost, uint64_t than) {
  const uint64_t margin = than / 24;
  return cost + (margin < 50 ? margin : 50) < than;
}

// rot_dot.hip's columns that go in a first call, the whole rounds; all n of them if
// the last round is better not taken apart, as where its loop would not split (56
// queries of 26 rotations x 46,052 entries 3,978 us, in two calls 4,351).
inline uint64_t rot_first_cols(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (room.cus < 8 || q == 0 || n == 0) return n;
  const uint64_t m = full_cols(n, rot_tiles(q * r, 256) * vecs, room) * kRotCols;
  if (m == 0 || m >= n || rot_splits(q * r, n - m, vecs, room) < 2) return n;
  const uint64_t apart = rot_cost(q, r, m, vecs, room) + rot_cost(q, r, n - m, vecs, room);
  return clearly_less(apart, rot_cost(q, r, n, vecs, room)) ? m : n;
}

inline uint64_t rot_rounds_cost(uint64_t q, uint32_t r, uint64_t n, uint32_t vecs, const DotRoom& room) {
  if (q == 0 || n == 0) return 0;
  const uint64_t m = rot_first_cols(q, r, n, vecs, room);
  return rot_cost(q, r, m, vecs, room) + rot_cost(q, r, n - m, vecs, room);
}

inline uint64_t pair_cost(uint64_t q, uint64_t cols, uint32_t vecs, const DotRoom& room) {
  const uint64_t tiles = xcd_cols(cols) * vecs * ((q + kPairQueries - 1) / kPairQueries);
  TileCost c = pair_tile_cost(q);
  if (tiles > uint64_t(room.cus) / 8) c.sparse -= 60;   // behind a full round
  return kLaunchCost + rounds_cost(tiles, c, room.cus);
}

struct RotPlan {
  uint32_t q;   // queries and columns of the pairs; the rest is rot_dot.hip's
  uint64_t n;
};

// Pairs take lists of 27 .. 31 consecutive rotations, ascending.
inline RotPlan rot_plan(uint32_t q_all, uint32_t r, const int8_t* rot, uint64_t n_all, uint32_t vecs,
                        const DotRoom& room) {
  const RotPlan none{0, 0};
  if (r < 27 || r > 31 || room.cus < 8) return none;
  for (uint32_t i = 1; i < r; ++i)
    if (rot[i] != rot[0] + int(i)) return none;
  RotPlan best = none;
  uint64_t least = rot_rounds_cost(q_all, r, n_all, vecs, room);
  const uint32_t over = q_all % kPairQueries;
  for (int less = 0; less < 2; ++less) {
    if (less && (over == 0 || over > kPairQueries / 2)) break;
    const uint32_t q = less ? q_all - over : q_all;
    if (q == 0) break;
    const uint64_t per = uint64_t(q + kPairQueries - 1) / kPairQueries * vecs, nt = (n_all + kRotCols - 1) / kRotCols;
    for (int part = 0; part < 2; ++part) {
      const uint64_t cols = part ? full_cols(n_all, per, room) : nt;
      if (cols == 0 || (part && cols >= nt)) break;
      const uint64_t n = cols * kRotCols < n_all ? cols * kRotCols : n_all;
      if (part && rot_splits(uint64_t(q) * r, n_all - n, vecs, room) < 2) break;
      const uint64_t cost = pair_cost(q, cols, vecs, room) + rot_rounds_cost(q, r, n_all - n, vecs, room) +
                            rot_rounds_cost(q_all - q, r, n_all, vecs, room);
      if (clearly_less(cost, least)) {
        least = cost;
        best = RotPlan{q, n};
      }
    }
  }
  return best;
}

}  // namespace imc
