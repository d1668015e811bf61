"""Log-normalisers of the full heads' rows from their statistics: added up four segments of a lane at a time, whatever the number of
loads in flight is.  The head's rows repeat every 128 tokens, so that a row's segments all have the same maximum and sum (read from the
kept statistics): every exponential is one, and the sum can be repeated in fp32 exactly.  The logarithm behind it need not round as
torch's does, so the two orders are told apart by the rows in which they give different results."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [50432, 131328, 180224])
def test_order_of_the_sum(V):
    import torch
    from paper_2410_17765_amd import binding
    T, d = 1024, 64
    print(f"V {V}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    H = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16)
    F = (torch.randn(128, d, generator=gen, device="cuda") * d ** -0.5).to(torch.bfloat16).repeat(V // 128, 1).reshape(1, 1, V, d).contiguous()
    G = torch.zeros(1, d, dtype=torch.bfloat16, device="cuda")
    X = torch.zeros(T, 1, dtype=torch.int32, device="cuda")
    ds = binding.make_desc(T, d, V, 1, 1, binding.BF16, binding.KEEP_LOGITS)
    size = binding.cp_head_full_ctx_bytes(ds)
    ctx, loss = torch.zeros(size, dtype=torch.uint8, device="cuda"), torch.empty(T, device="cuda")
    ws = torch.zeros(max(binding.cp_head_workspace_bytes(ds, binding.OP_FULL_LOSS_FWD), 256), dtype=torch.uint8, device="cuda")
    binding.cp_head_full_loss_fwd(ds, H, F, G, X, loss, ctx, ws)
    parts = V // 128
    lse = ctx[:4 * T].view(torch.float32)
    # the statistics lie before the kept logits, which end the buffer
    at = size - (2 * T * V + 255) // 256 * 256 - (8 * T * parts + 255) // 256 * 256
    stats = ctx[at:at + 8 * T * parts].view(torch.float32).view(T, parts, 2)
    assert torch.equal(stats, stats[:, :1].expand(T, parts, 2))
    lane = torch.arange(64, device="cuda")

    def normaliser(loads):
        total = torch.zeros(T, 64, device="cuda")
        for p0 in range(0, parts, 64 * loads):
            add = torch.zeros(T, 64, device="cuda")
            for lo in range(p0, min(p0 + 64 * loads, parts), 64):
                n = min(64, parts - lo)
                add[:, :n] += stats[:, lo:lo + n, 1]
            total += add
        for off in (32, 16, 8, 4, 2, 1):
            total = total + total[:, lane ^ off]
        return stats[:, 0, 0] + torch.log(total[:, 0])

    by_four, by_sixteen = normaliser(4), normaliser(16)
    assert (lse - by_four).abs().max() <= 4e-6
    told = by_four != by_sixteen
    assert int(told.sum()) >= 32
    assert int((lse == by_four)[told].sum()) > 2 * int((lse == by_sixteen)[told].sum())
