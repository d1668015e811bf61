"""Products whose last round of tiles is split along K: every product of the training step and of the full heads against
the oracle at sizes where the split has a ragged last part, rows and columns past the matrix, both outputs of the y
product, K-major operands that end inside a K-step; and the same step without scratch for it (least workspace)."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import rel_fro

pytestmark = pytest.mark.gpu

# T, d, V, n, r
CASES = [
    (300, 512, 3001, 2, 3),      # y 8 steps; dY 47; dU 29 (one tile row more than a multiple); dH 48; dW over 300 positions
    (1030, 320, 777, 1, 2),      # dW over 1030 positions: 17 steps, the last of 6 rows
    (70, 1024, 600, 4, 2),       # y 16 steps in 32 x 1 tiles; dH 128 steps
]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_training_step(oracle, shape):
    import torch
    from paper_2410_17765_amd import binding, head
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    cfg = synth.HeadConfig("split", T=T, d=d, V=V, n=n, r=r, targets="zipf")
    inp = synth.make_inputs(cfg)
    inp["X"][::7, n - 1] = -1
    ref = oracle.loss_bwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"])
    Hd, X = head.to_device(inp["H"], "bf16"), torch.from_numpy(inp["X"]).cuda()
    got = {}
    for flags in (0, binding.MIN_WORKSPACE):
        h = head.CpHead(inp["W"], inp["U"], inp["G"], dtype="bf16", flags=flags)
        assert flags or binding.cp_head_workspace_bytes(h.desc(T), binding.OP_LOSS_BWD) > 0
        h.loss_fwd(Hd, X)
        got[flags] = {k: v.cpu().numpy() for k, v in h.loss_bwd(Hd, X).items()}
        for k, v in ref.items():
            assert rel_fro(got[flags][k], v) <= 1e-2, (flags, k)
    # same operands: the sums differ by their order in fp32, and dY by the bf16 roundings that tip over with it (a share
    # of about sqrt(K) 2^-24 / 2^-8 of its elements, by 2^-8), and so much in what is formed from it
    for k in ref:
        assert rel_fro(got[0][k], got[binding.MIN_WORKSPACE][k]) <= 1e-3, k
