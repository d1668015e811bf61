"""The plain path's full heads: the products of all (s, a) share a launch, forward and backward, and agree with the oracle
where a launch holds many of them."""
import ctypes

import numpy as np
import pytest

from tests.helpers import rel_fro

pytestmark = pytest.mark.gpu


def launches(call):
    """Kernel launches that `call` records (it has run once before)."""
    import torch
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# T, d, V, n, r: few positions and many heads, rows and columns past the last tile, operands without 16-byte loads
@pytest.mark.parametrize("shape", [(4, 32, 64, 4, 4), (70, 45, 131, 3, 7), (2, 8, 9, 16, 16)], ids=lambda s: "x".join(map(str, s)))
def test_one_launch_for_all_heads(oracle, shape):
    import torch
    from paper_2410_17765_amd import head
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(9)
    H, F, G = (rng.standard_normal(s).astype(np.float32) for s in ((T, d), (n, r, V, d), (r, d)))
    X = rng.integers(0, V, (T, n), dtype=np.int32)
    X[::3, 0] = -1
    Hd, Xd = head.to_device(H, "fp32"), torch.from_numpy(X).cuda()
    h = head.CpFullHead(F, G, dtype="fp32")
    loss = h.loss_fwd(Hd, Xd).cpu().numpy()
    grads = {k: v.cpu().numpy() for k, v in h.loss_bwd(Hd, Xd).items()}
    ref = oracle.full_loss_fwd(H, F, G, X)
    # a few units in the last place of the loss; fp32 sums
    assert np.abs(loss - ref).max() <= 4e-6 * max(1.0, np.abs(ref).max())
    for k, v in oracle.full_loss_bwd(H, F, G, X).items():
        assert rel_fro(grads[k], v) <= 2e-5, (k, rel_fro(grads[k], v))
    one = head.CpFullHead(F[:1, :1], G[:1], dtype="fp32")
    X1 = Xd[:, :1].contiguous()
    one.loss_fwd(Hd, X1)
    one.loss_bwd(Hd, X1)
    assert launches(lambda: h.loss_fwd(Hd, Xd)) == launches(lambda: one.loss_fwd(Hd, X1)) <= 3
    assert launches(lambda: h.loss_bwd(Hd, Xd)) <= launches(lambda: one.loss_bwd(Hd, X1)) + 2      # split sums
