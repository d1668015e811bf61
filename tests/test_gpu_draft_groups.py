"""Draft calls that fit the static scratch array only without room for the logits of all drawn segments: a group of draws at
a time (whole rows of the batch; a part of one row's draws) against the same rows in calls that need no groups, bit for
bit."""
import pytest

pytestmark = pytest.mark.gpu

# T, d, V, n, r, rows per call without groups
CASES = [(7800, 64, 300, 4, 8, 1000), (8, 768, 100, 64, 62, 1)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_groups_of_draws(shape):
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r, few = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)

    def normal(*size, scale=1.0):
        out = torch.empty(size, dtype=torch.bfloat16, device="cuda")
        for part in out.view(-1).split(1 << 27):
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda") * scale)
        return out

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=4 * d ** -0.5)
    u = torch.rand((T, 1 + n), generator=gen, device="cuda")
    u[::7, 1:] = 1 - 2.0 ** -24
    ds = binding.make_desc(T, d, V, n, r, binding.BF16)
    need = binding.cp_head_workspace_bytes(ds, binding.OP_DRAFT)
    assert need <= binding.STATIC_SCRATCH_BYTES < need + T * n * r * (128 - (V + 255) // 256 * 8) * 4
    i32 = dict(dtype=torch.int32, device="cuda")
    alpha, tokens, logq = torch.empty(T, **i32), torch.empty((T, n), **i32), torch.empty(T, device="cuda")
    binding.cp_head_draft_sample_static(ds, H, W, U, G, u, alpha, tokens, logq)
    for lo in range(0, T, few):
        m = min(few, T - lo)
        sub = binding.make_desc(m, d, V, n, r, binding.BF16)
        ws = torch.empty(binding.cp_head_workspace_bytes(sub, binding.OP_DRAFT), dtype=torch.uint8, device="cuda")
        a, t, q = torch.empty(m, **i32), torch.empty((m, n), **i32), torch.empty(m, device="cuda")
        binding.cp_head_draft_sample(sub, H[lo:lo + m], W, U, G, u[lo:lo + m], a, t, q, ws)
        assert torch.equal(a, alpha[lo:lo + m]) and torch.equal(t, tokens[lo:lo + m]) and torch.equal(q, logq[lo:lo + m]), lo
    assert ((tokens >= 0) & (tokens < V)).all() and torch.isfinite(logq).all()
    # without the log-probability
    tokens2 = torch.empty((T, n), **i32)
    binding.cp_head_draft_sample_static(ds, H, W, U, G, u, alpha, tokens2, None)
    # another order of the sums where one launch picks them: a boundary of the running sum passes an ordinary uniform once in
    # thousands of draws, and one next to 1 far more often
    assert ((tokens2 >= 0) & (tokens2 < V)).all()
    ordinary = torch.arange(T, device="cuda") % 7 != 0
    assert (tokens != tokens2)[ordinary].sum() <= 1 + T * n // 1000
