"""Counts and statistic of eq. 10 on both sides of the lines at which the statistic gets a launch of its own (128 workgroups of
16 positions; T d max(r, 8) = 24 * 2^20), several calls on the same buffers: counts exactly those of the gate's arg-max, the statistic that of the counts."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 64, 3), (2048, 128, 8), (2049, 64, 8), (2050, 64, 17), (2000, 192, 64), (1536, 2048, 8), (1537, 2048, 2), (1536, 1024, 16), (1537, 1024, 16),
                                   (384, 1024, 64), (385, 1024, 64)], ids=lambda s: "x".join(map(str, s)))
def test_counts_and_statistic(shape):
    import torch
    from paper_2410_17765_amd import binding
    T, d, r = shape
    print(f"case {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    ds = binding.make_desc(T, d, 16, 1, r, binding.BF16, 0)
    counts = torch.full((r,), -1, dtype=torch.int64, device="cuda")
    laux, ws = torch.full((1,), float("nan"), device="cuda"), torch.empty(256, dtype=torch.uint8, device="cuda")
    for _ in range(20):
        # small whole numbers: the sums are exact, ties go to the first index
        H = torch.randint(-2, 3, (T, d), generator=gen, device="cuda").to(torch.bfloat16)
        G = torch.randint(-2, 3, (r, d), generator=gen, device="cuda").to(torch.bfloat16)
        binding.cp_head_aux_balance(ds, H, G, counts, laux, ws)
        gates = H.double().cpu() @ G.double().cpu().t()
        first = (gates == gates.max(dim=1, keepdim=True).values).to(torch.int8).argmax(dim=1)
        expected = torch.bincount(first, minlength=r)
        assert torch.equal(counts.cpu(), expected)
        stat = float(((expected.double() / T - 1.0 / r) ** 2).sum())
        assert abs(float(laux) - stat) <= 1e-6 * max(1.0, stat)
