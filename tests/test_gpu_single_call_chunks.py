"""The single training call against the pair of calls with kept logits where the batch is several chunks and the products'
last rounds are short enough to be split: the same loss bit for bit, and the same gradients (dU, whose chunks begin in other
rows where positions do not divide them, in another order of its fp32 sums)."""
import pytest

pytestmark = pytest.mark.gpu

# T, d, V, n, r: y in 23 x 45 tiles (11 in the last round) for the whole batch and 9 x 45 per chunk; chunks of 32768 rows, which
# 15 does not divide, or of whole positions
CASES = [(5888, 768, 65536, 3, 5), (5600, 768, 65536, 4, 4)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_same_results(shape):
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)

    def outputs():
        f32 = dict(dtype=torch.float32, device="cuda")
        return [torch.empty(s, **f32) for s in ((T,), (T, d), (n, r, d, d), (V, d), (r, d))]

    ds = binding.make_desc(T, d, V, n, r, binding.BF16, binding.KEEP_LOGITS)

    def scratch(*ops):
        return torch.empty(max(binding.cp_head_workspace_bytes(ds, op) for op in ops), dtype=torch.uint8, device="cuda")

    pair, single = outputs(), outputs()
    ctx, ws = torch.empty(binding.cp_head_ctx_bytes(ds), dtype=torch.uint8, device="cuda"), scratch(binding.OP_LOSS_FWD, binding.OP_LOSS_BWD)
    binding.cp_head_loss_fwd(ds, H, W, U, G, X, pair[0], ctx, ws)
    binding.cp_head_loss_bwd(ds, H, W, U, G, X, None, 1.0 / T, ctx, *pair[1:], ws)
    torch.cuda.synchronize()
    del ctx, ws
    binding.cp_head_loss_fwd_bwd(ds, H, W, U, G, X, None, 1.0 / T, *single, scratch(binding.OP_LOSS_FWD_BWD))
    for name, a, b in zip(("loss", "dH", "dW", "dU", "dG"), pair, single):
        if name != "dU":
            assert torch.equal(a, b), (name, float((a - b).norm() / b.norm()))
        else:
            assert (a - b).norm() <= 1e-6 * b.norm()          # fp32 sums of 90000 terms, some of them the other way round
