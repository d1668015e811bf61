"""The fine-tuning loss's forward call with the fp32 logits of a chunk of positions in memory (no flag), against the call that
multiplies U y a second time (least workspace) and against kept 16-bit logits: every rank of the path, vocabularies on both sides
of a tile of 256, of the teacher row that stays in registers (32768) and off the 8-column loads, one chunk and several."""
import pytest

pytestmark = pytest.mark.gpu

# T, d, V, n, r; the last: 3 GiB of fp32 logits are 12544 rows, the chunk a part of the batch
CASES = [(1, 64, 1, 1, 1), (37, 64, 255, 2, 1), (65, 128, 1001, 3, 2), (40, 64, 32771, 1, 4), (33, 64, 40001, 2, 8), (2500, 64, 64007, 1, 8)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_same_results(shape):
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    TZ = normal(T, n, V, scale=1.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    X[::5, n - 1] = -1
    f32 = dict(dtype=torch.float32, device="cuda")
    got = []
    for flags in (0, binding.MIN_WORKSPACE, binding.KEEP_LOGITS):
        ds = binding.make_desc(T, d, V, n, r, binding.BF16, flags)
        ctx = torch.empty(binding.cp_head_distill_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
        ws = torch.full((max(binding.cp_head_workspace_bytes(ds, op) for op in (binding.OP_DISTILL_FWD, binding.OP_DISTILL_BWD)),), 255,
                        dtype=torch.uint8, device="cuda")
        out = [torch.empty(s, **f32) for s in ((T,), (T, d), (n, r, d, d), (V, d), (r, d))]
        binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 0.9, 0.8, out[0], ctx, ws)
        binding.cp_head_distill_loss_bwd(ds, H, W, U, G, X, TZ, None, 1.0 / T, ctx, *out[1:], ws)
        torch.cuda.synchronize()
        got.append(out)
        del ctx, ws
    stored, product, kept = got
    # the same fp32 logits; S and KL are sums of V terms of one sign each up to cancellation in KL, in another order
    assert torch.isfinite(stored[0]).all()
    assert (stored[0] - product[0]).abs().max() <= 2e-5
    # 16-bit logits: 2^-11 relative to their block's maximum, averaged by the teacher's probabilities
    assert (stored[0] - kept[0]).abs().max() <= 5e-3
    for name, a, b in zip(("dH", "dW", "dU", "dG"), stored[1:], product[1:]):
        if name == "dG" and r == 1:
            # a softmax over one expert: dg = sum_k g_k (1 - R) / T is zero but for what R = sum_v p^c[v] misses 1 by, at most 4e-6
            # (p^c is exp of a difference of numbers up to 16 with errors of 2^-21), and dG is the sum of T of them times h
            assert max(float(a.norm()), float(b.norm())) <= n * 4e-6 * 1.5 * d ** 0.5
        else:                           # dz rounds to bf16: elements at a midpoint may tip over
            assert (a - b).norm() <= 1e-3 * b.norm(), name
