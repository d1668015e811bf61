"""The plain path's forward pass over several chunks of positions: chunks that end inside a tile of rows and in a rest, one
position with more head rows than a chunk asks for, dropped targets, both losses that use it."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import rel_fro
from tests.test_gpu_generic import run_loss

pytestmark = pytest.mark.gpu

# T, d, V, n, r, storage, flags (2: 256 rows of statistics at a time)
CASES = [
    (200, 50, 333, 3, 2, "fp32", 2),        # 42 positions at a time
    (150, 63, 1111, 2, 4, "bf16", 2),       # 32 at a time: whole tiles of rows, and a rest of 22
    (3, 20, 97, 5, 60, "fp32", 2),          # one at a time: 300 rows
    (1200, 16, 128256, 2, 2, "fp32", 0),    # 512 at a time: 2048 rows, all that 64 MiB hold at this vocabulary
]


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2410_17765_amd import binding, head
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return head


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_loss_and_gradients(gpu, oracle, shape):
    T, d, V, n, r, dtype, flags = shape
    cfg = synth.HeadConfig("chunks", T=T, d=d, V=V, n=n, r=r, dtype=dtype, targets="zipf")
    print(f"case {cfg} flags={flags}", flush=True)
    inp = synth.make_inputs(cfg)
    inp["X"][::5, n - 1] = -1
    dloss = synth.upstream_grad(T)
    loss, grads = run_loss(gpu, cfg, inp, dloss, flags=flags)
    ref = oracle.loss_fwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"])
    # as for one chunk: a few units in the last place of the loss, four fp32 sums in a chain
    assert np.abs(loss - ref).max() <= 4e-6 * max(1.0, np.abs(ref).max())
    for k, v in oracle.loss_bwd(inp["H"], inp["W"], inp["U"], inp["G"], inp["X"], dloss).items():
        assert rel_fro(grads[k], v) <= 2e-5, (k, rel_fro(grads[k], v))


def test_fine_tuning_loss(gpu, oracle):
    import torch
    cfg = synth.HeadConfig("chunks", T=200, d=50, V=333, n=3, r=2, dtype="fp32", targets="zipf")
    inp = synth.make_inputs(cfg)
    inp["X"][::5, 1] = -1
    tz = 1.5 * np.random.default_rng(3).standard_normal((cfg.T, cfg.n, cfg.V)).astype(np.float32)
    got = []
    for flags in (0, 2):
        h = gpu.CpHead(inp["W"], inp["U"], inp["G"], dtype="fp32", flags=flags)
        got.append(h.distill_loss_fwd(gpu.to_device(inp["H"], "fp32"), torch.from_numpy(inp["X"]).cuda(),
                                      torch.from_numpy(tz).cuda(), 0.9, 0.8).cpu().numpy())
    # the same sums over tiles of another width: a few units in the last place
    assert np.abs(got[0] - got[1]).max() <= 4e-6 * np.abs(got[0]).max()


# T, d, V, n, r: the forward pass of the full heads in chunks of 75 positions, and of 1024 and a rest
@pytest.mark.parametrize("shape", [(300, 24, 1, 1, 2), (1500, 8, 3, 1, 3)], ids=lambda s: "x".join(map(str, s)))
def test_full_heads(gpu, oracle, shape):
    import torch
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(8)
    H, F, G = (rng.standard_normal(s).astype(np.float32) for s in ((T, d), (n, r, V, d), (r, d)))
    X = rng.integers(0, V, (T, n), dtype=np.int32)
    h = gpu.CpFullHead(F, G, dtype="fp32")
    Hd, Xd = gpu.to_device(H, "fp32"), torch.from_numpy(X).cuda()
    loss = h.loss_fwd(Hd, Xd).cpu().numpy()
    ref = oracle.full_loss_fwd(H, F, G, X)
    assert np.abs(loss - ref).max() <= 4e-6 * max(1.0, np.abs(ref).max())
