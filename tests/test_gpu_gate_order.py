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


# T, d, r: less than one tile of 4 positions and 8 experts, one more than a tile of either, several groups of experts; fewer
# experts and more columns in flight, whole rounds of columns and a rest
@pytest.mark.parametrize("shape", [(1, 64, 2), (16, 128, 8), (37, 320, 9), (130, 1088, 64), (33, 1088, 2), (20, 704, 4), (9, 448, 3)], ids=lambda s: "x".join(map(str, s)))
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
    assert clear.sum() >= 0.7 * T or T == 1
    expect = g.max(axis=1) - g[:, 0]
    np.testing.assert_array_equal(loss[clear], expect[clear])


def weighted_sum_in_order(dg, H):
    """sum_t dg[t] H[t, :] over chunks of 512 positions, one fused multiply-add after the other, the chunks in turn."""
    total = np.zeros(H.shape[1], np.float32)
    for lo in range(0, len(dg), 512):
        acc = np.zeros(H.shape[1], np.float32)
        for g, h in zip(dg[lo:lo + 512], H[lo:lo + 512]):
            # a product has 32 bits: exact with 64 of them, like nearly every sum
            acc = (acc.astype(np.longdouble) + np.longdouble(g) * h.astype(np.longdouble)).astype(np.float32)
        total = total + acc
    return total


# one position, a batch of 16 positions and one more, a whole chunk of 512 and one more, three chunks; one and two groups
# of eight experts
@pytest.mark.parametrize("shape", [(1, 64, 2), (17, 192, 8), (512, 64, 3), (513, 128, 9), (1500, 64, 10)], ids=lambda s: "x".join(map(str, s)))
def test_gate_gradient(shape):
    import torch
    from paper_2410_17765_amd import head
    T, d, r = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(6)
    H = synth.bf16_round(rng.standard_normal((T, d)).astype(np.float32))
    H[:, 0] = 1                                       # as above: expert 0 explains every target
    W = np.zeros((1, r, d, d), np.float32)
    W[0, :, 0, 0] = -1024
    W[0, 0, 0, 0] = 1024
    U = np.zeros((2, d), np.float32)
    U[:, 0] = 1024, -1024
    h = head.CpHead(W, U, np.zeros((r, d), np.float32), dtype="bf16")
    Hd, X = head.to_device(H, "bf16"), torch.zeros((T, 1), dtype=torch.int32, device="cuda")
    up = rng.standard_normal(T).astype(np.float32)
    h.loss_fwd(Hd, X)
    dG = h.loss_bwd(Hd, X, torch.from_numpy(up).cuda())["dG"].cpu().numpy()
    # G = 0: all weights are one number next to 1/r, which only the device's exponential knows to the last bits
    one = np.float32(1) / np.float32(r)
    matches = []
    for ulps in range(-4, 5):
        w = (one.view(np.int32) + np.int32(ulps)).view(np.float32)
        if (weighted_sum_in_order(up * w, H) == dG[1:]).all():
            matches.append(w)
    assert len(matches) == 1
    np.testing.assert_array_equal(weighted_sum_in_order(up * (matches[0] - np.float32(1)), H), dG[0])
