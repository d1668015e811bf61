"""Logits of the plain path on both sides of each line between K-steps of 32 and of 16 (launches of 256, 512, 768, 1216, 2304 and 2560 tiles
of 128), against 64-bit torch: both storage types, widths that allow 16-byte loads and widths that do not, K with a part of a step left."""
import pytest

pytestmark = pytest.mark.gpu

V = 8192        # 64 tile columns
ROWS = [512, 513, 1024, 1025, 1536, 1537, 2432, 2433, 4608, 4609, 5120, 5121]


@pytest.mark.parametrize("d,dtype", [(100, "fp32"), (97, "fp32"), (100, "bf16"), (97, "bf16")])
@pytest.mark.parametrize("T", ROWS)
def test_loss_and_gradient(T, d, dtype):
    import torch
    from paper_2410_17765_amd import binding
    print(f"case T {T} d {d} {dtype}", flush=True)
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(store)

    H, G, W, U = normal(T, d), normal(1, d), normal(1, 1, d, d, scale=d ** -0.5), normal(V, d, scale=2 * d ** -0.5)
    X = torch.randint(0, V, (T, 1), generator=gen, device="cuda", dtype=torch.int32)
    ds = binding.make_desc(T, d, V, 1, 1, binding.BF16 if dtype == "bf16" else binding.FP32)
    ctx = torch.zeros(binding.cp_head_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(max(binding.cp_head_workspace_bytes(ds, op) for op in (binding.OP_LOSS_FWD, binding.OP_LOSS_BWD)), dtype=torch.uint8,
                     device="cuda")
    loss, dH = torch.empty(T, device="cuda"), torch.empty((T, d), device="cuda")
    binding.cp_head_loss_fwd(ds, H, W, U, G, X, loss, ctx, ws)
    binding.cp_head_loss_bwd(ds, H, W, U, G, X, None, 1.0, ctx, dH, None, None, None, ws)
    h, w, u = (t.double() for t in (H, W[0, 0], U))
    z = h @ w.t() @ u.t()
    expected = torch.logsumexp(z, 1) - z.gather(1, X.long()).squeeze(1)
    # fp32 sums of d terms of about 1 in each of two products, and of V exponentials
    assert (loss.double() - expected).abs().max() <= 4e-6 * expected.abs().max().clamp(min=1.0)
    p = torch.softmax(z, 1)
    p.scatter_add_(1, X.long(), torch.full((T, 1), -1.0, dtype=torch.float64, device="cuda"))
    dh = p @ u @ w
    assert (dH.double() - dh).norm() <= 1e-5 * dh.norm()
