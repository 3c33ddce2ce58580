"""The workgroup rules of the decode projections (csrc/gemv_plan.hpp), which are host code: compiled with the host
compiler behind a small C entry and set against timings taken on an MI355X."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21301_amd", "csrc")
SHIM = """
#include "gemv_plan.hpp"
extern "C" int rows(int N, int B, int cus, int head, int gate_up) {
  return nova::gemv_ring_rows(N, B, cus, head != 0, gate_up != 0);
}
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


# us of the LM head and the gate/up projection (K = 3584) as 128-row and as 64-row workgroups, the latter with the
# tail slices where the rule takes them: (weight rows, batch, CUs, 128 rows, 64 rows)
WIDE = [(HEAD, 1, 256, 180, 182), (HEAD, 8, 256, 188, 190), (HEAD, 32, 256, 203, 214), (HEAD, 1, 224, 184, 179),
        (HEAD, 8, 224, 192, 188), (HEAD, 32, 224, 212, 219), (HEAD, 1, 192, 190, 181), (HEAD, 8, 192, 200, 195),
        (HEAD, 4, 160, 200, 193), (HEAD, 16, 160, 221, 232), (HEAD, 1, 128, 222, 211), (HEAD, 4, 128, 231, 226),
        (HEAD, 12, 128, 247, 258), (HEAD, 1, 64, 365, 357), (HEAD, 8, 64, 389, 401), (HEAD, 32, 32, 904, 1081),
        (GATE_UP, 1, 64, 100, 92), (GATE_UP, 8, 64, 106, 102), (GATE_UP, 17, 64, 114, 124), (GATE_UP, 32, 64, 126, 144),
        (GATE_UP, 1, 32, 183, 168), (GATE_UP, 8, 32, 194, 189), (GATE_UP, 16, 32, 206, 211)]


@pytest.mark.parametrize("n,b,cus,wide,narrow", WIDE)
def test_rows_per_workgroup_against_timings(rules, n, b, cus, wide, narrow):
    rows = rules.rows(n, b, cus, n == HEAD, n == GATE_UP)
    assert (wide if rows == 128 else narrow) <= 1.01 * min(wide, narrow)


def test_ring_rows_need_two_rounds(rules):
    assert rules.rows(GATE_UP, 1, 76, 0, 1) == 0 and rules.rows(GATE_UP, 32, 256, 0, 1) == 0
    assert rules.rows(64 * 1021, 1, 64, 1, 0) == 0                  # no multiple of 128


# us of the gate/up projection as 64-row workgroups without and with tail slices: (batch, CUs, without, with)
TAIL = [(1, 256, 52.1, 48.5), (32, 256, 59.6, 55.1), (1, 192, 56.1, 48.5), (32, 192, 71.0, 62.3), (1, 160, 52.6, 51.9),
        (8, 160, 57.2, 56.6), (16, 160, 60.9, 62.2), (17, 160, 63.6, 66.1), (32, 160, 70.6, 75.6), (1, 128, 58.6, 55.8),
        (16, 128, 71.0, 70.3), (32, 128, 83.4, 84.4), (32, 96, 109.8, 102.2), (17, 32, 240.0, 236.5)]


@pytest.mark.parametrize("b,cus,without,sliced", TAIL)
def test_tail_slices_against_timings(rules, b, cus, without, sliced):
    assert (sliced if slices(rules, b, cus) > 1 else without) <= 1.01 * min(without, sliced)
