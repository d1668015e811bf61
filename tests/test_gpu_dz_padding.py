"""The logit gradients of a chunk are stored in whole blocks of 256 rows x 64 columns, and the products that read them run over
the padding too: no result may depend on what the workspace held before the call (a NaN there must not reach a gradient).
Rows and vocabularies on both sides of a block of 64, of 128 kept columns and of a tile of 256, over every loss."""
import pytest

pytestmark = pytest.mark.gpu

# T, d, V, n, r: 1, 63, 64, 111, 257 and 520 head rows (positions of the full heads: T)
CASES = [(1, 64, 1, 1, 1), (63, 64, 63, 1, 1), (64, 128, 65, 1, 1), (37, 64, 257, 3, 1), (257, 192, 129, 1, 1), (130, 64, 700, 2, 2)]


def outputs(kind, shape, fill):
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    def scratch(size):
        return torch.full((max(int(size), 256),), fill, dtype=torch.uint8, device="cuda")

    H, G = normal(T, d), normal(r, d, scale=d ** -0.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    X[::5, n - 1] = -1
    f32 = dict(dtype=torch.float32, device="cuda")
    loss, dH, dG = torch.empty(T, **f32), torch.empty((T, d), **f32), torch.empty((r, d), **f32)
    ds = binding.make_desc(T, d, V, n, r, binding.BF16, binding.KEEP_LOGITS if "keep" in kind else 0)

    def ws(*ops):
        return scratch(max(binding.cp_head_workspace_bytes(ds, op) for op in ops))

    if "full" in kind:
        F, dF = normal(n, r, V, d, scale=d ** -0.5), torch.empty((n, r, V, d), **f32)
        ctx, w = scratch(binding.cp_head_full_ctx_bytes(ds)), ws(binding.OP_FULL_LOSS_FWD, binding.OP_FULL_LOSS_BWD)
        binding.cp_head_full_loss_fwd(ds, H, F, G, X, loss, ctx, w)
        binding.cp_head_full_loss_bwd(ds, H, F, G, X, None, 1.0, ctx, dH, dF, dG, w)
        return loss, dH, dF, dG
    W, U = normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    dW, dU = torch.empty((n, r, d, d), **f32), torch.empty((V, d), **f32)
    if "tune" in kind:
        TZ = normal(T, n, V, scale=1.5)
        ctx, w = scratch(binding.cp_head_distill_ctx_bytes(ds)), ws(binding.OP_DISTILL_FWD, binding.OP_DISTILL_BWD)
        binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 0.9, 0.8, loss, ctx, w)
        binding.cp_head_distill_loss_bwd(ds, H, W, U, G, X, TZ, None, 1.0, ctx, dH, dW, dU, dG, w)
    elif kind == "single":
        binding.cp_head_loss_fwd_bwd(ds, H, W, U, G, X, None, 1.0, loss, dH, dW, dU, dG, ws(binding.OP_LOSS_FWD_BWD))
    else:
        ctx, w = scratch(binding.cp_head_ctx_bytes(ds)), ws(binding.OP_LOSS_FWD, binding.OP_LOSS_BWD)
        binding.cp_head_loss_fwd(ds, H, W, U, G, X, loss, ctx, w)
        binding.cp_head_loss_bwd(ds, H, W, U, G, X, None, 1.0, ctx, dH, dW, dU, dG, w)
    return loss, dH, dW, dU, dG


@pytest.mark.parametrize("kind", ["pair", "keep", "single", "full", "full keep", "tune", "tune keep"])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_scratch_contents_do_not_matter(shape, kind):
    import torch
    print(f"case {kind} {shape}", flush=True)
    clean, dirty = outputs(kind, shape, 0), outputs(kind, shape, 255)         # 0xFF..: NaN in every float type
    for a, b in zip(clean, dirty):
        assert torch.isfinite(a).all() and torch.equal(a, b)
