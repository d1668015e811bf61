"""Where the backward pass of the fine-tuning loss finds a token's teacher logits, checked on the CPU with the code that the kernels
compile (tests/teacher_rows_main.cpp): a chunk of one expert's rows holds more than 2^31 teacher logits from V = 65537 on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# M, V, r
CASES = [(32768, 65537, 1), (40000, 128256, 1), (100000, 151936, 1), (65536, 65600, 2), (262144, 128256, 8), (65536, 32000, 1), (3, 200000, 1)]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("teacher_rows") / "teacher_rows")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2410_17765_amd", "csrc"),
                    os.path.join(ROOT, "tests", "teacher_rows_main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe, *(str(x) for c in CASES for x in c)], check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_last_token_of_a_chunk(answers):
    assert len(answers) == len(CASES)
    for (M, V, r), (rows, start) in zip(CASES, answers):
        assert 1 <= rows <= M
        assert start == (rows // r - 1) * V
    # the cases reach what 32 bits do not
    assert sum(start + V > 2 ** 31 for (_, V, _), (_, start) in zip(CASES, answers)) >= 3
