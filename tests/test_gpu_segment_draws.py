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
