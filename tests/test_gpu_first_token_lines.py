"""First-token call on both sides of the line at which the mixture no longer forms the log-normalisers itself (2^21 pairs of statistics
read over the launch: B times the workgroups of 256 tokens times r times the segments), against the oracle; for segments of 64 columns
straight from memory, of 64 from the 64-row tile and of 128 from the 256-row tile."""
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_next_rows import gpu, test_first_token_logprob as check_first_token  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d, V, r
CASES = [(16, 64, 46000, 1), (16, 64, 46849, 1), (33, 64, 32000, 1), (33, 64, 32513, 1), (65, 64, 32000, 1), (65, 64, 32513, 1), (200, 64, 9000, 2)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, V, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("first_reads", T=T, d=d, V=V, n=1, r=r, targets="uniform", u_scale=2.0), 0)
