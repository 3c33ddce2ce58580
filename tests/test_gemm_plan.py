"""The tile plan of the encode and prefill GEMM (csrc/gemm_plan.hpp), which is host code: compiled with the
host compiler behind a small C entry and evaluated over the sizes of the stages' projections."""
import ctypes as C
import os
import subprocess
from collections import namedtuple

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21301_amd", "csrc")
SHIM = """
#include "gemm_plan.hpp"
extern "C" void plan(int M, int N, int K, int pos, int max_slices, unsigned long ws, int rows, int cols, int* v, double* us) {
  const nova::GemmPlan r = nova::plan_gemm(nova::GemmProblem{M, N, K, pos != 0, max_slices, ws, rows != 0, cols != 0});
  const int o[6] = {r.tile, r.slices, r.rows, r.cols, r.tile2, r.slices2};
  for (int i = 0; i < 6; ++i) v[i] = o[i];
  *us = r.us;
}
extern "C" int tiles(int* v) {
  for (int i = 0; i < nova::kGemmTileCount; ++i) v[2 * i] = nova::kGemmTiles[i].bm, v[2 * i + 1] = nova::kGemmTiles[i].bn;
  return nova::kGemmTileCount;
}
"""
STORE, GELU, RESID, POS, SWIGLU = range(5)
SLICE_FLOATS = 256 * 256 * 128
Plan = namedtuple("Plan", "tile slices rows cols tile2 slices2 us")
# the stages' projections: epilogue, V^T store, N, K; rows are patches (merge: a quarter of them) or prompt tokens
ENCODE = dict(qkv=(STORE, True, 3840, 1280), o=(RESID, False, 1280, 1280), up=(GELU, False, 5120, 1280),
              down=(RESID, False, 1280, 5120), merge=(STORE, False, 3584, 5120), patch=(POS, False, 1280, 640))
PREFILL = dict(qkv=(STORE, False, 4608, 3584), o=(RESID, False, 3584, 3584), gate_up=(SWIGLU, False, 37888, 3584),
               down=(RESID, False, 3584, 18944))


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = C.CDLL(str(so))
    v = (C.c_int * 32)()
    n = lib.tiles(v)
    lib.shapes = [(v[2 * i], v[2 * i + 1]) for i in range(n)]
    return lib


def plan(lib, proj, m, ws=None, slices=None, rows=None, cols=None):
    """The plan of one projection over m rows as the stages ask for it, or with one of the choices taken away."""
    epi, vt, n, k = proj
    sliced = epi != POS and not vt
    ws = max(SLICE_FLOATS, 4 * m * n // 2) if ws is None else ws
    v, us = (C.c_int * 6)(), C.c_double()
    lib.plan(m, n, k, int(epi == POS), (16 if sliced else 1) if slices is None else slices, C.c_ulong(ws),
             int(epi != POS) if rows is None else rows, int(sliced) if cols is None else cols, v, C.byref(us))
    return Plan(*v, us.value)


PROJECTIONS = [(f"encode_{k}", v) for k, v in ENCODE.items()] + [(f"prefill_{k}", v) for k, v in PREFILL.items()]


@pytest.mark.parametrize("proj", [p for _, p in PROJECTIONS], ids=[n for n, _ in PROJECTIONS])
def test_plans_fit(planner, proj):
    epi, vt, n, k = proj
    for m in [*range(1, 300, 7), *range(300, 42000, 331)]:
        for ws in (0, 3 * m * n, SLICE_FLOATS):
            r = plan(planner, proj, m, ws=ws)
            assert 0 <= r.tile < len(planner.shapes)
            bm, bn = planner.shapes[r.tile]
            first_n, rest_m, rest_n = r.cols or n, m - r.rows, n - r.cols
            assert first_n % bn == 0 and 0 <= r.rows < m and 0 <= r.cols < n and not (r.rows and r.cols)
            assert r.rows % 8 == 0                       # a V^T store goes by eights of tokens
            if r.rows or r.cols:
                assert r.slices == 1 and rest_n % planner.shapes[r.tile2][1] == 0
            slices = r.slices2 if r.rows or r.cols else r.slices
            steps = -(-(k // 64) // slices)
            assert slices == 1 or (not vt and epi != POS and slices * rest_m * rest_n <= ws and (slices - 1) * steps < k // 64)
            if epi == POS:
                assert not r.rows and not r.cols
            if vt:
                assert not r.cols


@pytest.mark.parametrize("proj", [p for n, p in PROJECTIONS if p[0] != POS], ids=[n for n, p in PROJECTIONS if p[0] != POS])
def test_plan_is_the_least_estimate(planner, proj):
    """No choice that could run instead has a lower estimate than the plan."""
    for m in [*range(64, 4100, 97), *range(4104, 41480, 56)]:
        r = plan(planner, proj, m)
        for kw in (dict(rows=0), dict(cols=0), dict(rows=0, cols=0), dict(slices=1), dict(slices=1, rows=0, cols=0)):
            assert r.us <= plan(planner, proj, m, **kw).us * (1 + 1e-12), (m, kw)
