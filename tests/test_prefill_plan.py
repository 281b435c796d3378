"""The rule that picks a prefill call's form, compiled from the library's own
header by the host compiler."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import test_gpu_prefill as gpu
from conftest import ROOT

SHIM = """
#include "prefill_plan.hpp"
extern "C" int plan(int n, int H, int G, int total_rows, int max_rows, long long capacity) {
  const sm::PrefillPlan p = sm::plan_prefill(n, H, G, total_rows, max_rows, capacity);
  return p.few ? -p.splits : p.splits;
}
"""


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    """plan(requests, kv heads, group, rows, most rows, capacity): the groups of waves, or "few"."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2609_27233_amd", "csrc"), str(d / "plan.cpp"), "-o",
                    str(d / "plan.so")], check=True, timeout=120)
    f = C.CDLL(str(d / "plan.so")).plan
    f.argtypes = [C.c_int] * 5 + [C.c_longlong]
    return lambda *a: {-4: "few"}.get(f(*a), f(*a))


def _capacity(lens, bs):
    return (max(-(-L // bs) for L in lens) + 2) * bs           # as test_gpu_prefill's cache


@pytest.mark.parametrize("case", range(len(gpu.SPLIT_CASES)))
def test_sizes_of_the_gpu_tests_take_the_form_they_name(plan, case):
    Hq, H, D, bs, lens, ms, form = gpu.SPLIT_CASES[case]
    ms = list(lens) if ms is None else ms
    assert plan(len(lens), H, Hq // H, sum(ms), max(ms), _capacity(lens, bs)) == form


def test_gpu_tests_reach_every_kernel():
    assert {(c[2], c[6]) for c in gpu.SPLIT_CASES} == {(D, f) for D in (64, 128) for f in (1, 2, 4, "few")}


@pytest.mark.parametrize("Hq,H", [(32, 8), (8, 8), (28, 4), (64, 8), (16, 4)])
def test_the_capacity_matters_to_long_whole_prompts_only(plan, Hq, H):
    """A cache larger than a prompt needs changes nothing for calls of few
    workgroups, and a bound on the context only lets longer prompts split."""
    G = Hq // H
    for n in (1, 2, 4):
        for rows in (1, 8, 16, 32, 64, 100, 128, 200, 400, 639, 640, 900, 1200, 1500, 2048, 4096):
            tight, loose = plan(n, H, G, n * rows, rows, rows), plan(n, H, G, n * rows, rows, 1 << 20)
            if tight != loose:
                assert (tight, loose) == (2, 1) and rows >= 640
            if n * rows * Hq <= 256 * 64:                       # a quarter of the units or less: split whatever the cache
                assert loose in (4, "few")
            assert (loose == "few") == (loose != 1 and loose != 2 and rows * G <= 128)
