"""The order of the fp32 sums in the gate of the matrix-core path, bit for bit: log-weights differ from one order to the
next by some units in the last place, enough to tip bf16 roundings further down."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth

pytestmark = pytest.mark.gpu


def gates_in_order(H, G):
    """G h with 64 running sums over the columns l, l + 64, ..., added up 32, 16, ... 1 apart (the products of two bfloat16
    are exact in fp32)."""
    T, d = H.shape
    lane = np.arange(64)
    out = np.empty((T, G.shape[0]), np.float32)
    for a, g in enumerate(G):
        s = np.zeros((T, 64), np.float32)
        for k in range(0, d, 64):
            s += H[:, k:k + 64] * g[None, k:k + 64]
        for off in (32, 16, 8, 4, 2, 1):
            s = s + s[:, lane ^ off]
        out[:, a] = s[:, 0]
    return out


# T, d, r: less than one tile of 4 positions and 8 experts, one more than a tile of either, several groups of experts
@pytest.mark.parametrize("shape", [(1, 64, 2), (16, 128, 8), (37, 320, 9), (130, 1088, 64)], ids=lambda s: "x".join(map(str, s)))
def test_log_weights(shape):
    import torch
    from paper_2410_17765_amd import head
    T, d, r = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(5)
    H = synth.bf16_round(8 * rng.standard_normal((T, d)).astype(np.float32))
    G = synth.bf16_round(8 * rng.standard_normal((r, d)).astype(np.float32))
    # the first column of H makes expert 0 certain of token 0 and the others certain of token 1 (log-probability -2^21),
    # all in exact arithmetic, so that the loss of token 0 is the log-weight of expert 0
    H[:, 0] = 1
    W = np.zeros((1, r, d, d), np.float32)
    W[0, :, 0, 0] = -1024
    W[0, 0, 0, 0] = 1024
    U = np.zeros((2, d), np.float32)
    U[:, 0] = 1024, -1024
    h = head.CpHead(W, U, G, dtype="bf16")
    loss = h.loss_fwd(head.to_device(H, "bf16"), torch.zeros((T, 1), dtype=torch.int32, device="cuda")).cpu().numpy()
    g = gates_in_order(H, G)
    top = np.sort(g, axis=1)
    # where the largest gate leads by 20, the sum of exponentials is 1 and the log-weight g_0 - max g, exactly
    clear = top[:, -1] - top[:, -2] > 20
    assert clear.sum() >= 0.8 * T or r == 2
    expect = g.max(axis=1) - g[:, 0]
    np.testing.assert_array_equal(loss[clear], expect[clear])
