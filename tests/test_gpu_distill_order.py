"""The fine-tuning loss's forward call gives the same bits whether it passes over the fp32 logits of a chunk of positions (no flag)
or multiplies U y a second time (least workspace): what it leaves for the backward call and the loss are sums of the same terms in
the same order.  Every rank of the path, vocabularies on both sides of 64, of a sub-tile of 128 columns, of 32 and 64 sub-tiles (4096, 8192) and of
the lines between the forms of the teacher's log-normalisers (512, 8192) and what they hold in registers (32768); one chunk of positions and several."""
import pytest

pytestmark = pytest.mark.gpu

# T, d, V, n, r; the last: 3 GiB of fp32 logits are 12544 rows, the chunk a part of the batch
CASES = [(1, 64, 1, 1, 1), (37, 64, 255, 2, 1), (100, 64, 512, 4, 8), (65, 128, 2049, 3, 2), (40, 64, 4096, 1, 8), (40, 64, 4097, 1, 8), (40, 64, 8192, 1, 4), (40, 64, 8193, 1, 4), (33, 64, 32771, 2, 8),
         (20, 64, 65537, 1, 2), (2500, 64, 64007, 1, 8)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_same_bits(shape):
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    TZ = normal(T, n, V, scale=1.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    X[::5, n - 1] = -1
    got = []
    for flags in (0, binding.MIN_WORKSPACE):
        ds = binding.make_desc(T, d, V, n, r, binding.BF16, flags)
        ctx = torch.zeros(binding.cp_head_distill_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
        ws = torch.full((binding.cp_head_workspace_bytes(ds, binding.OP_DISTILL_FWD),), 255, dtype=torch.uint8, device="cuda")
        loss = torch.empty(T, dtype=torch.float32, device="cuda")
        binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 0.9, 0.8, loss, ctx, ws)
        torch.cuda.synchronize()
        got.append((loss, ctx))
        del ws
    assert torch.isfinite(got[0][0]).all()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
