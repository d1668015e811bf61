"""The fine-tuning loss's forward call in a workspace that holds the statistics of a second product but no chunk of fp32 logits: the same
bits as in the workspace that the query reports, and nothing written behind the smaller one."""
import pytest

from paper_2410_17765_amd import binding
from tests.test_distill_refused import second_product_bytes

pytestmark = pytest.mark.gpu

# T, d, V, n, r: one row; a y product whose last round is split along d; 3 GiB of logits are fewer rows than the batch has
CASES = [(1, 64, 200, 1, 1), (100, 1024, 1000, 1, 4), (2500, 64, 64007, 1, 8)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_same_bits(shape):
    import torch
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    TZ = normal(T, n, V, scale=1.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    ds = binding.make_desc(T, d, V, n, r, binding.BF16)
    need, least = binding.cp_head_workspace_bytes(ds, binding.OP_DISTILL_FWD), second_product_bytes(*shape)
    got = []
    for size in (need, least):
        whole = torch.full((size + 4096,), 255, dtype=torch.uint8, device="cuda")
        ctx, loss = torch.zeros(binding.cp_head_distill_ctx_bytes(ds), dtype=torch.uint8, device="cuda"), torch.empty(T, device="cuda")
        binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 0.9, 0.8, loss, ctx, whole[:size])
        assert (whole[size:] == 255).all()
        got.append((loss, ctx))
        del whole
    assert least < need
    assert torch.isfinite(got[0][0]).all()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
