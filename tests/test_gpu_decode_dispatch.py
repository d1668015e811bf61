"""The decoding calls on both sides of each line of their dispatch, against the oracle.
First token: z straight from memory for up to 16 / 32 head rows and 65536 tokens, on tiles beyond; the log-normalisers inside the
mixture for up to 4096 pairs of statistics (r times the segments), in a launch of their own beyond.
Sequential: up to 64, 1024 and 2048 segments with at most eight experts; more segments, more experts."""
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_next_rows import gpu, run_sequential, test_first_token_logprob as check_first_token  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d, V, r
FIRST = [(1, 64, 1, 1), (1, 128, 63, 1), (2, 64, 64, 8), (17, 64, 65, 1), (4, 576, 129, 8), (3, 64, 1000, 11), (4, 64, 32768, 8), (4, 64, 32769, 8),
         (2, 128, 65536, 2), (2, 128, 65537, 2), (1, 64, 65600, 16), (33, 64, 300, 1), (1, 192, 5000, 33)]
# T, d, V, n, r
SEQUENTIAL = [(2, 64, 64, 3, 8), (3, 128, 4096, 2, 8), (3, 64, 4097, 2, 7), (9, 64, 8193, 2, 8), (2, 64, 65537, 2, 8), (1, 64, 131073, 2, 3),
              (2, 64, 500, 2, 9)]


@pytest.mark.parametrize("shape", FIRST, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, V, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("first_line", T=T, d=d, V=V, n=2, r=r, targets="uniform", u_scale=2.0), 0)


@pytest.mark.parametrize("shape", SEQUENTIAL, ids=lambda s: "x".join(map(str, s)))
def test_sequential(gpu, oracle, shape):  # noqa: F811
    T, d, V, n, r = shape
    run_sequential(gpu, oracle, synth.HeadConfig("seq_line", T=T, d=d, V=V, n=n, r=r, targets="uniform", u_scale=4.0), 0)
