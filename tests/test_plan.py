"""The host-side rules of the dot calls (csrc/plan.h), compiled here without a GPU."""
import ctypes
import os
import subprocess

import pytest

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
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, out = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2405_04463_amd", "csrc"), str(src), "-o", str(out)], check=True)
    return ctypes.CDLL(str(out))


def test_parts_are_lent_to_one_stream_only(plan):
    u = ctypes.c_void_p
    assert plan.lends(0, u(0), u(5), 0, 0) == 1          # nobody's yet
    assert plan.lends(1, u(5), u(5), 0, 0) == 1
    assert plan.lends(1, u(5), u(6), 0, 0) == 0
    assert plan.lends(1, u(0), u(0), 0, 0) == 1          # the default stream
    for owned, of in ((0, 0), (1, 2)):
        assert plan.lends(owned, u(of), u(2), 1, 0) == 0  # one handle, a stream in every thread
        assert plan.lends(owned, u(of), u(2), 0, 1) == 0  # captured


def test_splits_stay_within_the_loop_the_cus_and_the_scratch(plan):
    f = lambda *a: plan.splits(ctypes.c_uint64(a[0]), a[1], a[2], ctypes.c_uint64(a[3]), ctypes.c_size_t(a[4]), a[5])  # noqa: E731
    assert f(16, 1, 32, 1000, 1 << 25, 256) == 16
    assert f(2, 1, 32, 1000, 1 << 25, 256) == 32         # the loop's pieces
    assert f(2, 2, 80, 1000, 1 << 25, 256) == 80
    assert f(2, 1, 32, 1 << 20, 1 << 25, 256) == 8       # 32 MiB of u32 sums
    assert f(200, 1, 32, 1000, 1 << 25, 256) == 1
    assert f(2, 1, 32, 1000, 0, 256) == 1                # not lent
    assert f(2, 1, 32, 1 << 40, 1 << 25, 256) == 1


def test_rows_of_a_rotation_tile(plan):
    """The fewest rows at which all tiles run at once, a column tile's on one of 8 XCDs."""
    f = lambda rows, nt, vecs, cus=256: plan.tile_rows(ctypes.c_uint64(rows), ctypes.c_uint64(nt), vecs, cus)  # noqa: E731
    assert f(31, 8, 2) == 64 and f(247, 1, 2) == 64
    assert f(1024, 1, 2) == 64 and f(1025, 1, 2) == 128   # 32 CUs of one XCD: 16 tiles a vector
    assert f(1025, 1, 1) == 64 and f(2049, 8, 1) == 128
    assert f(2080, 8, 2) == 192 and f(2080, 9, 2) == 256
    assert f(104, 40, 1) == 64 and f(260, 40, 2) == 128
    assert f(200, 129, 2) == 256 and f(128, 65, 2) == 128 and f(128, 129, 2) == 256
    assert f(31, 8, 2, 8) == 256 and f(31, 8, 2, 16) == 64 and f(31, 8, 2, 0) == 256
