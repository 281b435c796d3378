"""The rule that picks a merge call's GEMM, compiled from the library's own
header by the host compiler."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import test_gpu_gemm_shapes as shapes
from conftest import ROOT

TILES = ["32x32", "32x64", "64x64", "96x64", "128x64", "160x64", "192x64", "256x128", "256x256", "plain", "skinny"]

SHIM = """
#include "gemm_plan.hpp"
extern "C" void plan(int M, int N, int K, int f32, int aligned, int *out) {
  const sm::GemmPlan p = sm::plan_gemm(M, N, K, f32 != 0, aligned != 0);
  out[0] = p.kind, out[1] = p.rows, out[2] = p.kind2;
}
"""


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    """plan(rows, d, f32, aligned): the tiles as text, "a+b" for a call cut in two, and the rows of the first."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2609_27233_amd", "csrc"), str(d / "plan.cpp"), "-o",
                    str(d / "plan.so")], check=True, timeout=120)
    lib = C.CDLL(str(d / "plan.so"))

    def f(rows, width, f32=False, aligned=True):
        out = (C.c_int * 3)()
        lib.plan(rows, width, width, int(f32), int(aligned), out)
        first = TILES[out[0]]
        return (first if out[1] == rows else first + "+" + TILES[out[2]]), out[1]

    return f


@pytest.mark.parametrize("d", [256, 768, 3584, 8192])
def test_operands_off_16_bytes_take_the_plain_loads(plan, d):
    for rows in (1, 16, 63, 64):
        assert plan(rows, d, aligned=False) == ("skinny", rows)
    for rows in (65, 300, 40000):
        assert plan(rows, d, aligned=False) == ("plain", rows)
    for rows in (1, 64, 300, 40000):
        assert plan(rows, d, f32=True, aligned=False) == ("plain", rows)


@pytest.mark.parametrize("d,rows,tile,f32", [(*c, False) for c in shapes.BF16 + shapes.SPANS] + [
    (*c, True) for c in shapes.F32])
def test_sizes_of_the_gpu_tests_take_the_kernels_they_name(plan, d, rows, tile, f32):
    assert plan(rows, d, f32)[0] == tile


def test_gpu_tests_reach_every_kernel():
    for cases, kinds in ((shapes.BF16, TILES), (shapes.F32, TILES[:7] + ["plain"]), (shapes.SPANS, TILES)):
        assert {t for _, _, tile in cases for t in tile.split("+")} == set(kinds)
    for cases in (shapes.BF16, shapes.SPANS):               # and calls cut in two
        assert any("+" in tile for _, _, tile in cases)


def test_plan_covers_the_rows_and_fits_the_width(plan):
    """Every call gets all its rows, whole tiles of columns, and a first part of whole row tiles."""
    for d in range(256, 8193, 256):
        for rows in (1, 2, 31, 32, 33, 64, 65, 127, 300, 999, 2049, 4097, 10001, 65535, 200003, 8 << 20):
            for f32 in (False, True):
                tile, first = plan(rows, d, f32)
                parts = tile.split("+")
                assert 0 < first <= rows and (len(parts) == 2) == (first < rows)
                for t in parts:
                    if "x" in t:
                        bm, bn = map(int, t.split("x"))
                        assert d % bn == 0 and not (f32 and bm == 256)
                if len(parts) == 2:
                    assert first % int(parts[0].split("x")[0]) == 0
                if "skinny" in parts:
                    assert rows <= 64 and not f32
