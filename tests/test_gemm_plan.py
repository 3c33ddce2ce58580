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
extern "C" void plan(int M, int N, int K, int epi, int cus, int max_slices, unsigned long ws, int rows, int cols,
                     int* v, double* us) {
  const nova::GemmPlan r = nova::plan_gemm(nova::GemmProblem{M, N, K, epi, cus, max_slices, ws, rows != 0, cols != 0});
  const int o[6] = {r.tile, r.slices, r.rows, r.cols, r.tile2, r.slices2};
  for (int i = 0; i < 6; ++i) v[i] = o[i];
  *us = r.us;
}
extern "C" int f32_small(int M, int N, int cus) { return nova::gemm_f32_small(M, N, cus); }
extern "C" int tiles(int* v) {
  for (int i = 0; i < nova::kGemmTileCount; ++i) {
    v[2 * i] = nova::kGemmTiles[i].bm;
    v[2 * i + 1] = nova::kGemmTiles[i].bn;
  }
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


def plan(lib, proj, m, ws=None, slices=None, rows=None, cols=None, cus=256):
    """The plan of one projection over m rows as the stages ask for it, or with one of the choices taken away."""
    epi, vt, n, k = proj
    sliced = epi != POS and not vt
    ws = max(SLICE_FLOATS, 4 * m * 4608 if proj in PREFILL.values() else 2 * m * n) if ws is None else ws
    v, us = (C.c_int * 6)(), C.c_double()
    lib.plan(m, n, k, epi, cus, (16 if sliced else 1) if slices is None else slices, C.c_ulong(ws),
             int(epi != POS) if rows is None else rows, int(sliced) if cols is None else cols, v, C.byref(us))
    return Plan(*v, us.value)


PROJECTIONS = [(f"encode_{k}", v) for k, v in ENCODE.items()] + [(f"prefill_{k}", v) for k, v in PREFILL.items()]


@pytest.mark.parametrize("proj", [p for _, p in PROJECTIONS], ids=[n for n, _ in PROJECTIONS])
def test_plans_fit(planner, proj):
    epi, vt, n, k = proj
    for m in [*range(1, 300, 7), *range(300, 42000, 331)]:
        cus = (256, 224, 104, 32, 8)[m % 5]
        for ws in (0, 3 * m * n, SLICE_FLOATS):
            r = plan(planner, proj, m, ws=ws, cus=cus)
            assert 0 <= r.tile < len(planner.shapes)
            bm, bn = planner.shapes[r.tile]
            first_n, rest_m, rest_n = r.cols or n, m - r.rows, n - r.cols
            assert first_n % bn == 0 and 0 <= r.rows < m and 0 <= r.cols < n and not (r.rows and r.cols)
            assert r.rows % 8 == 0                       # a V^T store goes by eights of tokens
            if r.rows or r.cols:
                assert r.slices == 1 and rest_n % planner.shapes[r.tile2][1] == 0
            slices = r.slices2 if r.rows or r.cols else r.slices
            steps = -(-(k // 64) // slices)
            if slices > 1:
                assert not vt and epi != POS and slices * rest_m * rest_n <= ws and (slices - 1) * steps < k // 64
            if epi == POS:
                assert not r.rows and not r.cols
            if vt:
                assert not r.cols


# Single launches timed on an MI355X (us, by (tile, K slices), the fastest first), at sizes where a split into two
# launches is slower or not possible.  One 1008x1008 image's MLP up projection takes 86 us as two launches.
# Compute units of the stream first.
TIMED = [
    (256, ENCODE["up"], 5184, {(7, 1): 81.8, (6, 1): 92.7, (5, 1): 95.8, (4, 1): 96.8}),
    (256, ENCODE["up"], 2304, {(7, 1): 44.5, (6, 1): 45.9, (3, 1): 47.2, (5, 1): 49.3}),
    (256, ENCODE["o"], 5184, {(4, 1): 26.8, (5, 1): 27.5, (6, 1): 28.0, (3, 1): 30.5}),
    (256, ENCODE["down"], 5184, {(5, 1): 76.4, (4, 1): 76.5, (6, 1): 80.0, (7, 2): 82.7}),
    (256, ENCODE["down"], 1600, {(4, 3): 37.0, (5, 3): 37.9, (2, 1): 38.3, (6, 3): 39.2}),
    (256, ENCODE["down"], 312, {(2, 5): 17.0, (3, 8): 19.5}),
    (256, ENCODE["down"], 360, {(3, 8): 18.0, (0, 1): 19.7}),
    (256, ENCODE["merge"], 576, {(4, 3): 36.8, (5, 3): 37.0, (2, 1): 39.8, (6, 3): 39.8}),
    (256, ENCODE["patch"], 1600, {(2, 1): 9.5, (1, 1): 9.8, (3, 1): 10.6, (0, 1): 12.5}),
    (256, ENCODE["patch"], 5184, {(4, 1): 17.1, (6, 1): 17.4, (5, 1): 17.4, (3, 1): 19.8, (7, 1): 24.8}),
    (256, ENCODE["patch"], 13416, {(6, 1): 41.7, (5, 1): 44.2, (4, 1): 44.3, (3, 1): 45.8, (7, 1): 49.2}),
    (256, ENCODE["patch"], 20736, {(7, 1): 51.6, (6, 1): 56.6, (5, 1): 59.0}),
    (256, ENCODE["patch"], 41472, {(7, 1): 120.0, (5, 1): 126.2, (4, 1): 126.4, (6, 1): 126.7}),
    (256, PREFILL["qkv"], 203, {(3, 3): 20.0, (4, 6): 21.6, (5, 6): 22.0, (4, 5): 22.3}),
    (256, PREFILL["qkv"], 1, {(0, 3): 10.7, (0, 2): 11.0, (0, 7): 11.8}),
    (256, PREFILL["qkv"], 6, {(0, 3): 11.0, (0, 7): 12.1}),
    (256, PREFILL["down"], 1500, {(7, 3): 179.7, (7, 6): 200.4, (4, 3): 209.2}),
    (224, PREFILL["gate_up"], 1500, {(7, 1): 345.7, (5, 1): 441.1, (4, 1): 442.2}),
    (224, PREFILL["down"], 1500, {(7, 5): 208.1, (7, 2): 215.5, (7, 8): 219.9}),
    (192, ENCODE["qkv"], 5184, {(7, 1): 63.6, (5, 1): 78.2, (6, 1): 78.8}),
    (160, ENCODE["down"], 5184, {(7, 3): 103.6, (7, 1): 111.5, (7, 4): 118.9}),
    (128, PREFILL["qkv"], 768, {(4, 1): 50.8, (5, 1): 52.1, (7, 2): 55.0}),
    (96, ENCODE["o"], 1024, {(3, 1): 16.1, (1, 1): 21.7, (2, 1): 22.5}),
    (64, ENCODE["o"], 1024, {(4, 1): 23.4, (5, 1): 23.9, (6, 1): 24.4}),
    (32, ENCODE["down"], 1024, {(7, 3): 99.0, (7, 4): 108.8, (7, 1): 116.1}),
]


@pytest.mark.parametrize("cus,proj,m,us", TIMED)
def test_plan_against_timings(planner, cus, proj, m, us):
    """The plan runs as one launch that takes at most 9% longer than the fastest timed one."""
    r = plan(planner, proj, m, cus=cus)
    assert not r.rows and not r.cols
    assert us.get((r.tile, r.slices), 1e9) <= 1.09 * min(us.values()), r


@pytest.mark.parametrize("name", [n for n, p in PROJECTIONS if p[0] != POS])
def test_plan_is_the_least_estimate(planner, name):
    """No choice that could run instead has a lower estimate than the plan."""
    proj = dict(PROJECTIONS)[name]
    for m in [*range(64, 4100, 97), *range(4104, 41480, 56)]:
        r = plan(planner, proj, m)
        for kw in (dict(rows=0), dict(cols=0), dict(rows=0, cols=0), dict(slices=1), dict(slices=1, rows=0, cols=0)):
            assert r.us <= plan(planner, proj, m, **kw).us * (1 + 1e-12), (m, kw)


# fp32 activations, us: (CUs, rows, N, 32x64 tiles, 128x128 tiles)
F32 = [(256, 256, 1280, 12.1, 37.2), (256, 2304, 1280, 35.9, 45.3), (256, 1024, 3840, 47.3, 45.9),
       (256, 3200, 1280, 179.0, 159.5), (256, 1024, 5120, 59.3, 89.7), (256, 4096, 1280, 58.6, 86.8),
       (256, 2304, 3840, 95.3, 126.0), (256, 2304, 5120, 124.9, 133.7), (256, 3200, 3840, 136.4, 128.6),
       (256, 15552, 1280, 244.9, 214.6), (256, 10368, 5120, 627.6, 565.0), (128, 256, 3840, 27.8, 38.0),
       (128, 4000, 512, 14.7, 11.8), (128, 3200, 1280, 80.6, 86.1), (128, 2304, 5120, 210.5, 261.1),
       (64, 256, 3840, 47.5, 37.5), (64, 1024, 1280, 53.0, 81.0), (64, 4096, 1280, 180.8, 209.4)]


@pytest.mark.parametrize("cus,m,n,small,large", F32)
def test_f32_tiles_against_timings(planner, cus, m, n, small, large):
    assert (small if planner.f32_small(m, n, cus) else large) <= 1.03 * min(small, large)
