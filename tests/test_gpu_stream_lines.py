"""z of 17 to 32 head rows straight from memory or on tiles, on both sides of each line of that choice, against the oracle: 32768
columns (one round of workgroups); beyond it widths from 2048 on, and there two rounds that are seven eighths full (448 workgroups of
128 columns)."""
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_next_rows import gpu, run_sequential, test_first_token_logprob as check_first_token  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d, V, r
CASES = [(17, 64, 32768, 1), (32, 64, 32769, 1), (17, 1984, 57345, 1), (17, 2048, 57216, 1), (17, 2048, 57217, 1), (17, 2048, 65409, 1)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, V, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("stream_line", T=T, d=d, V=V, n=1, r=r, targets="uniform", u_scale=2.0), 0)


@pytest.mark.parametrize("shape", [(4, 64, 32768, 1, 8), (4, 64, 32769, 1, 8)], ids=lambda s: "x".join(map(str, s)))
def test_sequential(gpu, oracle, shape):  # noqa: F811
    T, d, V, n, r = shape
    run_sequential(gpu, oracle, synth.HeadConfig("stream_line", T=T, d=d, V=V, n=n, r=r, targets="uniform", u_scale=4.0), 0)
