"""The index maps of the GEMM launches, checked on the CPU: the header that holds them has no HIP dependency, so
the same code the kernels compile is built here with g++ and run over a sweep of shapes (tests/tile_walk_main.cpp:
workgroup -> tile: every tile exactly once, grid size, the XCDs in step over the columns; the block-by-block operand
layout: a bijection with contiguous 8-column pieces and contiguous 256 x 64 blocks)."""
import os
import subprocess

import pytest

from tests.test_gpu_split_round import FULL_HEADS, TRAINING_STEPS, full_heads_products, training_products

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tile_walk") / "tile_walk")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2410_17765_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tile_walk_main.cpp"), "-o", exe], check=True)
    return exe


def test_tile_walk_and_blocked_layout(exe):
    out = subprocess.run([exe], check=False, capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.startswith("ok ")


def test_the_split_cases_are_split(exe):
    """What the GPU tests of split last rounds say about their sizes: (whole tiles before the split ones, parts) per product."""
    for cases, products in ((TRAINING_STEPS, training_products), (FULL_HEADS, full_heads_products)):
        for shape, expected in cases.items():
            for name, sizes in products(*shape).items():
                out = subprocess.run([exe, *map(str, sizes)], check=True, capture_output=True, text=True).stdout
                first, tail, parts = map(int, out.split())
                assert (first, parts) == expected.get(name, (first, 1)), (shape, name, out)
    # between them: every product, the residual of y included, next to whole tiles and alone
    split = [(name, plan) for cases in (TRAINING_STEPS, FULL_HEADS) for e in cases.values() for name, plan in e.items()]
    assert {name for name, _ in split} >= {"y", "dY", "dU", "dH", "dW", "full dH", "full dF"}
    assert {name for name, (first, _) in split if first} >= {"y", "dY", "dU"}
