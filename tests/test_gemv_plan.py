"""The workgroup rules of the decode projections (csrc/gemv_plan.hpp), which are host code: compiled with the host
compiler behind a small C entry and set against timings taken on an MI355X."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21301_amd", "csrc")
SHIM = """
#include "gemv_plan.hpp"
extern "C" int wide(int N, int cus) { return nova::gemv_wide(N, cus); }
extern "C" int tail(int N, int K, int B, int cus, int counters, unsigned long floats) {
  return nova::gemv_tail(N, K, B, cus, counters, floats);
}
"""
HEAD, GATE_UP, K = 152064, 37888, 3584
COUNTERS, FLOATS = 112, 1 << 22


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemv")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return C.CDLL(str(so))


def slices(lib, b, cus, n=GATE_UP, k=K, counters=COUNTERS, floats=FLOATS):
    return lib.tail(n, k, b, cus, counters, C.c_ulong(floats))


def test_tail_slices_fit(rules):
    """Every slice holds K, the tiles fit the counters and the partials the workspace."""
    for cus in range(8, 257, 8):
        for n in range(64, 40000, 1664):
            for k in (256, 512, 1024, 1280, 3584, 18944):
                for counters, floats in ((0, 1 << 22), (32, 1 << 22), (112, 1 << 22), (112, 30000)):
                    s = slices(rules, 7, cus, n, k, counters, floats)
                    tiles, chunks = n // 64, k // 256
                    assert 1 <= s <= 4
                    if s > 1:
                        assert tiles >= cus and 0 < tiles % cus <= counters and s * (tiles % cus) * 64 * 7 <= floats
                        assert (s - 1) * -(-chunks // s) < chunks
