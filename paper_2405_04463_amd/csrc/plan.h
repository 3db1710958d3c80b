// plan.h -- host-side rules of the dot calls that need no GPU: who may use a
// context's scratch, and how a K loop is split.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace imc {

// Which stream may use a context's parts scratch: the first whose call splits a
// K loop, for the life of the context, since only one stream's calls are known
// to run in order.  Not lent to captured calls (a graph may be replayed beside
// eager calls) nor to the per-thread default stream, whose one handle names
// another stream in every thread.
struct PartsOwner {
  bool owned = false;
  uintptr_t stream = 0;
  bool lends(uintptr_t to, bool per_thread, bool capturing) const {
    return !capturing && !per_thread && (!owned || stream == to);
  }
  void take(uintptr_t by) {
    owned = true;
    stream = by;
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

}  // namespace imc
