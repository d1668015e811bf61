"""The fp32 matrix-core products of the plain path at the edges of their tiles: every tile edge (128, 64, 32) in every launch,
split sums, several chunks, partial K-steps, rows and columns past the last whole tile, operands that allow 16-byte loads
and operands that do not."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import rel_fro
from tests.test_gpu_generic import run_loss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2410_17765_amd import binding, head
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return head


# T, d, V, n, r, storage: {tile edge of the logits, of the launch of dY and dU, of the launch of dH, dW and dG; K-splits; chunks},
# one where nothing is said (checked on the CPU)
CASES = {
    (200, 128, 3333, 4, 4, "fp32"): {"z": 128, "chunk": 64, "dY": 8, "dU": 2, "weights": 32, "dH": 8},
    # no operand aligned, bf16 widened on the way in
    (257, 333, 3001, 2, 3, "bf16"): {"z": 64, "chunk": 64, "weights": 32},
    # one expert
    (1024, 48, 256, 1, 1, "fp32"): {"z": 32, "chunk": 32, "dU": 4, "weights": 32, "dW": 4, "dG": 4},
    # few rows, a K-step of 4 left over
    (33, 260, 5000, 1, 2, "fp32"): {"z": 32, "chunk": 32, "dY": 4, "weights": 32},
    # odd everything
    (130, 97, 1501, 3, 5, "fp32"): {"z": 128, "chunk": 32, "weights": 32, "dH": 4},
    # less than one tile, less than one K-step
    (1, 4, 1, 1, 1, "fp32"): {"z": 32, "chunk": 32, "weights": 32},
    # 128-wide tiles in every launch, K-major operands among them: M, N and K past the last whole tile or K-step, with 16-byte
    # loads and (odd sizes) without
    (301, 500, 2100, 4, 8, "fp32"): {"z": 128, "chunk": 128, "dY": 2, "dU": 2, "weights": 128, "dH": 16},
    (301, 501, 2099, 4, 8, "fp32"): {"z": 128, "chunk": 128, "dY": 2, "dU": 2, "weights": 128, "dH": 16},
    (1300, 380, 1020, 4, 4, "fp32"): {"z": 128, "chunk": 128, "dU": 8, "weights": 128, "dH": 4, "dW": 4, "dG": 4},
    # two chunks: split parts of dU added to what is there
    (4300, 44, 8191, 2, 2, "fp32"): {"chunks": 2, "z": 128, "chunk": 64, "dU": 2, "weights": 32, "dW": 16, "dG": 16},
    (400, 380, 4500, 4, 4, "fp32"): {"z": 128, "chunk": 128, "dU": 8, "weights": 64, "dH": 4},
}


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_loss_and_gradients(gpu, oracle, shape):
    T, d, V, n, r, dtype = shape
    cfg = synth.HeadConfig("tiles", T=T, d=d, V=V, n=n, r=r, dtype=dtype, targets="zipf")
    print(f"case {cfg}", flush=True)
    inp = synth.make_inputs(cfg)
    if T > 1:
        inp["X"][::5, n - 1] = -1
    dloss = synth.upstream_grad(T)
    loss, grads = run_loss(gpu, cfg, inp, dloss, flags=1)
    ref = oracle.loss_fwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"])
    # log-sum-exp over fp32 logits: a few units in the last place of the loss
    assert np.abs(loss - ref).max() <= 4e-6 * max(1.0, np.abs(ref).max())
    gref = oracle.loss_bwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"], dloss)
    # an fp32 sum of K random terms is off by about sqrt(K) 2^-24, 8e-6 at the largest K here (17200); four such sums in a chain
    for k, v in gref.items():
        if np.linalg.norm(v) == 0:
            assert np.abs(grads[k]).max() <= 1e-6, k
        else:
            assert rel_fro(grads[k], v) <= 2e-5, (k, rel_fro(grads[k], v))
