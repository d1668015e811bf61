"""First-token call on both sides of the line between one and two blocks of W in flight (8192 columns of y; beyond them widths past 2048),
with an odd number of blocks of 64 columns for a wavefront among them, against the oracle."""
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_next_rows import gpu, test_first_token_logprob as check_first_token  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d, r
CASES = [(3, 1024, 7), (3, 1024, 8), (16, 1216, 7), (2, 2048, 4), (1, 2112, 4)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("y_blocks", T=T, d=d, V=300, n=1, r=r, targets="uniform", u_scale=2.0), 0)
