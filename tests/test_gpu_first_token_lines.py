"""First-token call on both sides of the lines at which the mixture no longer forms the log-normalisers itself, against the oracle; for
segments of 64 columns straight from memory, of 64 from the 64-row tile and of 128 from the 256-row tile.  2^21 pairs of statistics
read over the launch (B times the workgroups of 256 tokens times r times the segments): the first two pairs of cases.  Workgroups: 2048 of
them, 1024 with more than four experts."""
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_next_rows import gpu, test_first_token_logprob as check_first_token  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d, V, r
CASES = [(8, 64, 32768, 4), (8, 64, 32769, 4), (16, 64, 23040, 4), (16, 64, 23297, 4), (16, 64, 32768, 1), (16, 64, 32769, 1), (64, 64, 8192, 1), (64, 64, 8193, 1),
         (16, 64, 46849, 1), (128, 64, 4096, 2), (128, 64, 4097, 2), (2, 64, 1000, 5), (16, 64, 16384, 5), (16, 64, 16385, 5), (200, 64, 9000, 2)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, V, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("first_reads", T=T, d=d, V=V, n=1, r=r, targets="uniform", u_scale=2.0), 0)
