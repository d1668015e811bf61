"""The tiles and split sums that the GPU tests of the plain path's products say they use, from the same header that the
library plans with (it has no HIP dependency: built here with g++), and the bound on the split sums' scratch."""
import os
import subprocess

import pytest

from tests.test_gpu_f32_tiles import CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("f32_plan") / "f32_plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2410_17765_amd", "csrc"),
                    os.path.join(ROOT, "tests", "f32_plan_main.cpp"), "-o", exe], check=True)

    def run(*shape):
        out = subprocess.run([exe, *map(str, shape)], check=True, capture_output=True, text=True).stdout
        return {k: int(v) for k, v in (pair.split("=") for pair in out.split())}
    return run


def test_cases_are_planned_as_stated(plan):
    seen = set()
    for (T, d, V, n, r, _), stated in CASES.items():
        got = plan(T, d, V, n, r)
        for key, value in got.items():
            assert value == stated.get(key, 1), ((T, d, V, n, r), key, got)
        seen |= {(launch, got[launch]) for launch in ("z", "chunk", "weights")}
        seen |= {(product, "split") for product in ("dY", "dU", "dH", "dW", "dG") if got[product] > 1}
        if got["chunks"] > 1 and got["dU"] > 1:
            seen.add("split dU over several chunks")
    assert seen == {(launch, edge) for launch in ("z", "chunk", "weights") for edge in (128, 64, 32)} | \
        {(product, "split") for product in ("dY", "dU", "dH", "dW", "dG")} | {"split dU over several chunks"}


def test_split_sums_are_bounded(plan):
    for T in (1, 33, 500, 4000, 16384, 1 << 20):
        for d in (16, 500, 4096):
            for V in (500, 32000, 128256):
                for n, r in ((1, 1), (4, 8), (16, 64)):
                    p = plan(T, d, V, n, r)
                    rows = min(max((1 << 27) // ((V + 3) // 4 * 4) // r * r, r), T * n * r)
                    parts = {"dY": rows * d, "dU": V * d, "dH": T * d, "dW": n * r * d * d, "dG": r * d}
                    for launch in (("dY", "dU"), ("dH", "dW", "dG")):
                        assert sum(p[k] * parts[k] * 4 for k in launch if p[k] > 1) <= 128 << 20, (T, d, V, n, r, p)
