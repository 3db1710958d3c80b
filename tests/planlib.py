"""csrc/plan.h compiled for the host (a helper of the tests, not a test module)."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "plan.h"
extern "C" {
int lends(int owned, uintptr_t stream, uintptr_t to, int per_thread, int capturing) {
  imc::PartsOwner o;
  o.owned = owned;
  o.stream = stream;
  return o.lends(to, per_thread, capturing);
}
unsigned splits(uint64_t tiles, unsigned per_cu, unsigned units, uint64_t outputs, size_t bytes, int cus) {
  return imc::dot_splits(tiles, per_cu, units, outputs, bytes, cus);
}
unsigned tile_rows(uint64_t rows, uint64_t nt, unsigned vecs, int cus) { return imc::rot_tile_rows(rows, nt, vecs, cus); }
unsigned lead_tiles(uint64_t rows, uint64_t tiles, int cus) { return imc::rot_lead_tiles(rows, tiles, cus); }
unsigned rot_splits(uint64_t rows, uint64_t n, unsigned vecs, size_t bytes, int cus, int galois) {
  return imc::rot_splits(rows, n, vecs, imc::DotRoom{bytes, cus, imc::rot_segs(galois)});
}
uint64_t rot_cost(uint64_t q, unsigned r, uint64_t n, unsigned vecs, size_t bytes, int cus, int galois) {
  return imc::rot_cost(q, r, n, vecs, imc::DotRoom{bytes, cus, imc::rot_segs(galois)});
}
uint64_t first_cols(uint64_t q, unsigned r, uint64_t n, unsigned vecs, size_t bytes, int cus, int galois) {
  return imc::rot_first_cols(q, r, n, vecs, imc::DotRoom{bytes, cus, imc::rot_segs(galois)});
}
void plan(unsigned q, unsigned r, const int8_t* rot, uint64_t n, unsigned vecs, size_t bytes, int cus, int galois,
          uint64_t out[2]) {
  const imc::RotPlan p = imc::rot_plan(q, r, rot, n, vecs, imc::DotRoom{bytes, cus, imc::rot_segs(galois)});
  out[0] = p.q;
  out[1] = p.n;
}
}
"""
SCRATCH = 32 << 20      # a context's scratch for the parts of split loops


class Plan:
    """Calls into the compiled header; room = (scratch bytes, CUs)."""

    def __init__(self, folder):
        src, out = os.path.join(folder, "shim.cpp"), os.path.join(folder, "shim.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                        os.path.join(ROOT, "paper_2405_04463_amd", "csrc"), src, "-o", out], check=True)
        L = self.L = ctypes.CDLL(out)
        u64, u32, sz, i = ctypes.c_uint64, ctypes.c_uint, ctypes.c_size_t, ctypes.c_int
        L.lends.argtypes = [i, ctypes.c_void_p, ctypes.c_void_p, i, i]
        L.splits.argtypes = [u64, u32, u32, u64, sz, i]
        L.tile_rows.argtypes = [u64, u64, u32, i]
        L.lead_tiles.argtypes = [u64, u64, i]
        L.rot_splits.argtypes = [u64, u64, u32, sz, i, i]
        L.rot_cost.argtypes = [u64, u32, u64, u32, sz, i, i]
        L.rot_cost.restype = u64
        L.first_cols.argtypes, L.first_cols.restype = L.rot_cost.argtypes, u64
        L.plan.argtypes = [u32, u32, ctypes.c_char_p, u64, u32, sz, i, i, ctypes.POINTER(u64)]

    def plan(self, q, rot, n, vecs=2, galois=False, scratch=SCRATCH, cus=256):
        """(queries, columns) that go in pairs of rotations."""
        out = (ctypes.c_uint64 * 2)()
        self.L.plan(q, len(rot), bytes(s & 0xFF for s in rot), n, vecs, scratch, cus, galois, out)
        return tuple(out)
