"""The gate kernels of the matrix-core path (log-softmax of G h, arg-max counts, gate gradient) at the edges of their
tiles: 16 positions and 16 experts per product, 4 x 64 columns per round, 128 positions and 512 columns per partial sum."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import rel_fro

pytestmark = pytest.mark.gpu

# T, d, r
CASES = [(1, 64, 1), (15, 64, 16), (17, 320, 17), (129, 576, 9), (300, 1088, 33), (257, 512, 64), (8209, 128, 5)]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_gate_counts_and_gradient(oracle, shape):
    import torch
    from paper_2410_17765_amd import head
    T, d, r = shape
    print(f"case {shape}", flush=True)
    cfg = synth.HeadConfig("gate", T=T, d=d, V=16, n=1, r=r)
    inp = synth.make_inputs(cfg)
    h = head.CpHead(inp["W"], inp["U"], inp["G"], dtype="bf16")
    Hd, X = head.to_device(inp["H"], "bf16"), torch.from_numpy(inp["X"]).cuda()
    counts, laux = h.aux_balance(Hd)
    h.loss_fwd(Hd, X)
    dG = h.loss_bwd(Hd, X)["dG"].cpu().numpy()
    c_o, l_o = oracle.aux_balance(inp["H"].astype(np.float64), inp["G"].astype(np.float64))
    # gates are N(0, 1): two of a position's agree to the 2^-20 of an fp32 sum once in about 10^5 positions
    assert np.abs(counts.cpu().numpy() - c_o).sum() <= 2 * (T // 50000)
    assert abs(float(laux[0]) - l_o) <= 1e-6 * max(1.0, l_o)
    g_o = oracle.loss_bwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"])["dG"]
    # r = 1 has no gate gradient; else the loss path's bound for bf16 operands
    assert np.abs(dG).max() <= 1e-6 if r == 1 else rel_fro(dG, g_o) <= 1e-2
