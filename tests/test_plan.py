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
