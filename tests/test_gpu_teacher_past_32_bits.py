"""Backward call of the fine-tuning loss where a chunk's teacher logits pass 2^31 elements (32768 tokens of one expert, V = 65600),
against the same call in chunks of 256 rows (least workspace), which never get there."""
import pytest

pytestmark = pytest.mark.gpu


def test_chunk_of_more_than_2_to_31_teacher_logits():
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = 32768, 64, 65600, 1, 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)

    def normal(*size, scale=1.0):
        out = torch.empty(size, dtype=torch.bfloat16, device="cuda")
        flat = out.view(-1)
        for lo in range(0, flat.numel(), 1 << 28):
            part = flat[lo:lo + (1 << 28)]
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda") * scale)
        return out

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    TZ = normal(T, n, V, scale=1.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    got = []
    for flags in (0, binding.MIN_WORKSPACE):
        ds = binding.make_desc(T, d, V, n, r, binding.BF16, flags)
        ctx = torch.zeros(binding.cp_head_distill_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
        ws = torch.empty(max(binding.cp_head_workspace_bytes(ds, op) for op in (binding.OP_DISTILL_FWD, binding.OP_DISTILL_BWD)),
                         dtype=torch.uint8, device="cuda")
        loss, dH, dG = torch.empty(T, device="cuda"), torch.empty((T, d), device="cuda"), torch.empty((r, d), device="cuda")
        dW = torch.empty((n, r, d, d), device="cuda")
        binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 0.9, 0.8, loss, ctx, ws)
        binding.cp_head_distill_loss_bwd(ds, H, W, U, G, X, TZ, None, 1.0, ctx, dH, dW, None, dG, ws)
        torch.cuda.synchronize()
        got.append((loss, dH, dW))
        del ctx, ws
    assert torch.equal(got[0][0], got[1][0])
    # the same logit gradients; fp32 sums over V in another split, rounded to bf16 once: elements at a midpoint may tip over
    for a, b in zip(got[0][1:], got[1][1:]):
        assert (a - b).norm() <= 1e-3 * b.norm()
    # and row by row where the offsets are largest
    tail = slice(T - 256, T)
    assert (got[0][1][tail] - got[1][1][tail]).norm() <= 1e-3 * got[1][1][tail].norm()
