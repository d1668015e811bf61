"""Draws of both decoding calls at the edges of the segment kernels: 16 tokens and 16 experts per product, 8 x 4 blocks
of 64 columns per round, 64- and 128-column segments, more segments than the 1024 threads that search them; and on both
sides of the limits of the streamed y product: 16 positions, 8 of them beyond 32768 columns."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import check_draft, check_sequential

pytestmark = pytest.mark.gpu

# T, d, V, n, r
CASES = [(1, 64, 17, 1, 1), (3, 320, 1000, 2, 16), (2, 576, 66001, 2, 17), (1, 2112, 4097, 3, 2), (5, 128, 513, 17, 5),
         (70, 64, 257, 2, 33), (16, 448, 100, 1, 4), (17, 64, 100, 1, 4), (8, 1088, 65, 1, 31), (9, 1088, 65, 1, 31)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_draws(oracle, shape):
    import torch
    from paper_2410_17765_amd import head
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    cfg = synth.HeadConfig("segment", T=T, d=d, V=V, n=n, r=r, targets="uniform", u_scale=4.0)
    inp = synth.make_inputs(cfg)
    args = (inp["H"], inp["W"], inp["U"], inp["G"])
    h = head.CpHead(inp["W"], inp["U"], inp["G"], dtype="bf16")
    Hd = head.to_device(inp["H"], "bf16")
    u = synth.uniforms(T, n)
    # both checks hold every draw to the oracle's running sum: inside its band, and the log-probability at the drawn tuple
    alpha, tokens, logq = (t.cpu().numpy() for t in h.draft_sample(Hd, torch.from_numpy(u).cuda()))
    stats = check_draft(oracle, *args, u, alpha, tokens, logq, round_y=True, logq_atol=2e-3)
    print(f"  {stats}", flush=True)
    us = np.ascontiguousarray(u[:, 1:])
    tokens, logq = (t.cpu().numpy() for t in h.draft_sample_sequential(Hd, torch.from_numpy(us).cuda()))
    stats = check_sequential(oracle, *args, us, tokens, logq, logq_atol=2e-3)
    print(f"  {stats}", flush=True)
    # a uniform that every running sum passes, one that hardly any does
    for value in (0.0, float(np.nextafter(np.float32(1), np.float32(0)))):
        _, tok, lq = h.draft_sample(Hd, torch.full((T, 1 + n), value, device="cuda"))
        tok_s, lq_s = h.draft_sample_sequential(Hd, torch.full((T, n), value, device="cuda"))
        for x, q in ((tok, lq), (tok_s, lq_s)):
            assert ((x >= 0) & (x < V)).all() and torch.isfinite(q).all()


# 64 to 1024 draws and one on either side, 64- and 128-column segments, partial ones, more than one step of the contraction per lane
@pytest.mark.parametrize("shape", [(64, 64, 17, 1, 1), (70, 576, 1000, 2, 3), (16, 320, 257, 4, 1), (512, 64, 65, 2, 2), (33, 1088, 65, 2, 2), (63, 64, 700, 1, 1),
                                   (205, 64, 33, 5, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_draws_without_log_probability(oracle, shape):
    """The token of a draw lies in the oracle's band, as with the log-probability asked for."""
    import torch
    from paper_2410_17765_amd import binding, head
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    cfg = synth.HeadConfig("segment", T=T, d=d, V=V, n=n, r=r, targets="uniform", u_scale=4.0)
    inp = synth.make_inputs(cfg)
    h = head.CpHead(inp["W"], inp["U"], inp["G"], dtype="bf16")
    Hd = head.to_device(inp["H"], "bf16")
    ds = h.desc(T)
    ws = torch.empty(binding.cp_head_workspace_bytes(ds, binding.OP_DRAFT), dtype=torch.uint8, device="cuda")

    def sample(u, logq):
        alpha, tokens = torch.empty(T, dtype=torch.int32, device="cuda"), torch.full((T, n), -7, dtype=torch.int32, device="cuda")
        binding.cp_head_draft_sample(ds, Hd, h.W, h.U, h.G, u, alpha, tokens, logq, ws)
        return alpha.cpu().numpy(), tokens.cpu().numpy()

    u = synth.uniforms(T, n)
    ud, logq = torch.from_numpy(u).cuda(), torch.empty(T, dtype=torch.float32, device="cuda")
    a1, t1 = sample(ud, logq)
    a0, t0 = sample(ud, None)
    np.testing.assert_array_equal(a0, a1)
    # the two differ where fp32 sums in another order move a boundary of the running sum across u: once in thousands of draws
    assert (t0 != t1).sum() <= 1 + T * n // 1000
    check_draft(oracle, inp["H"], inp["W"], inp["U"], inp["G"], u, a0, t0, None, round_y=True)
    for value in (0.0, float(np.nextafter(np.float32(1), np.float32(0)))):
        _, tok = sample(torch.full((T, 1 + n), value, device="cuda"), None)
        assert ((tok >= 0) & (tok < V)).all()
