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

}  // namespace imc
