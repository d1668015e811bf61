"""First-token call, against the oracle.  On both sides of the lines at which the statistics come from a pass over the stored logits: 65 to 96
rows of 256-row tiles, and 5 * 2^19 logits up to 2048 rows, with one and several segments of 4096 columns.  On both sides of the lines at which the mixture no longer forms the log-normalisers itself; for
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
APART = [(65, 64, 1, 1), (65, 64, 4097, 1), (12, 128, 12289, 8), (97, 64, 27024, 1), (97, 64, 27025, 1), (64, 64, 5120, 8), (64, 64, 5121, 8), (200, 64, 515, 3)]


@pytest.mark.parametrize("shape", CASES + APART, ids=lambda s: "x".join(map(str, s)))
def test_first_token(gpu, oracle, shape):  # noqa: F811
    T, d, V, r = shape
    check_first_token(gpu, oracle, synth.HeadConfig("first_reads", T=T, d=d, V=V, n=1, r=r, targets="uniform", u_scale=2.0), 0)


@pytest.mark.parametrize("T,V", [(2048, 1280), (2048, 1281), (2049, 130)])
def test_many_rows(T, V):
    """2048 rows, and one more: y of small whole numbers is exact, so that no rounding of it can tip over."""
    import torch
    from paper_2410_17765_amd import binding
    d = 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + V)
    H, W = (torch.randint(-1, 2, size, generator=gen, device="cuda").to(torch.bfloat16) for size in ((T, d), (1, 1, d, d)))
    U = (torch.randn(V, d, generator=gen, device="cuda") / 16).to(torch.bfloat16)
    G = torch.zeros(1, d, dtype=torch.bfloat16, device="cuda")
    ds = binding.make_desc(T, d, V, 1, 1, binding.BF16)
    logp = torch.empty(T, V, device="cuda")
    ws = torch.empty(binding.cp_head_workspace_bytes(ds, binding.OP_FIRST_TOKEN), dtype=torch.uint8, device="cuda")
    binding.cp_head_first_token_logprob(ds, H, W, U, G, logp, ws)
    expected = torch.log_softmax(H.double() @ W[0, 0].double().t() @ U.double().t(), dim=1)
    # fp32 sums of 64 products and of V exponentials, logits of up to 30
    assert (logp.double() - expected).abs().max() <= 2e-5
