"""Products whose last round of tiles is split along K: the training step against the oracle at sizes where every one of its
products is split in some case, alone and next to whole tiles in one launch, with ragged last parts, rows and columns past
the matrix, both outputs of the y product, K-major operands that end inside a K-step; dU added up over several chunks; the
full heads' products; and the same steps without scratch for it (least workspace).  Which product is split at which size
is checked on the CPU."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.helpers import rel_fro

pytestmark = pytest.mark.gpu


def training_products(T, d, V, n, r):
    """M, N, K of the step's products if the batch is one chunk."""
    M, nrd = T * n * r, n * r * d
    return {"y": (T, nrd, d), "dY": (M, d, -(-V // 64) * 64), "dU": (V, d, -(-M // 64) * 64), "dH": (T, d, nrd), "dW": (nrd, d, T)}


def full_heads_products(T, d, V, n, r):
    return {"full dH": (T, d, -(-V // 64) * 64), "full dF": (V, d, -(-T // 64) * 64)}


# T, d, V, n, r: {product: (whole tiles before the split ones, parts)}, the others are not split
TRAINING_STEPS = {
    (300, 512, 3001, 2, 3): {"dY": (0, 6), "dU": (0, 5), "dH": (0, 8)},
    (1030, 320, 777, 1, 2): {"dU": (0, 7), "dW": (0, 4)},           # dW over 1030 positions: 17 K-steps, the last of 6 rows
    (70, 1024, 600, 4, 2): {"dH": (0, 16)},
    (1500, 768, 1000, 3, 5): {"y": (256, 3), "dY": (256, 4), "dU": (0, 16), "dH": (0, 10)},
    (600, 448, 33001, 1, 2): {"dY": (0, 16), "dU": (256, 4), "dH": (0, 3)},
}
FULL_HEADS = {(1500, 768, 1000, 1, 2): {"full dH": (0, 4), "full dF": (0, 4)}}


@pytest.mark.parametrize("shape", TRAINING_STEPS, ids=lambda s: "x".join(map(str, s)))
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
    got, loss = {}, {}
    for flags in (0, binding.MIN_WORKSPACE):
        h = head.CpHead(inp["W"], inp["U"], inp["G"], dtype="bf16", flags=flags)
        loss[flags] = h.loss_fwd(Hd, X).cpu().numpy()
        got[flags] = {k: v.cpu().numpy() for k, v in h.loss_bwd(Hd, X).items()}
        for k, v in ref.items():
            assert rel_fro(got[flags][k], v) <= 1e-2, (flags, k)
    # target logits come from y and its residual, which leave out nothing of it but 2^-17; in the log-normalisers the bf16
    # roundings that tip over (a share of 1e-3 of y, by 2^-8) move single logits by 1e-4 and their sums by less
    assert np.abs(loss[0] - loss[binding.MIN_WORKSPACE]).max() <= 3e-4
    # same operands: the sums differ by their order in fp32, and dY by the bf16 roundings that tip over with it (a share
    # of about sqrt(K) 2^-24 / 2^-8 of its elements, by 2^-8), and so much in what is formed from it
    for k in ref:
        assert rel_fro(got[0][k], got[binding.MIN_WORKSPACE][k]) <= 1e-3, k


def test_accumulation_over_chunks():
    """dU over two chunks of the batch, whole tiles and split ones in both launches (65 x 4 tiles): against the sums of the
    least-workspace call, 256 rows at a time and never split."""
    import torch
    from paper_2410_17765_amd import binding
    T, d, V, n, r = 8200, 1024, 16640, 4, 4              # 131200 rows, 126976 of them in the first chunk
    print(f"case {(T, d, V, n, r)}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def normal(*size, scale=1.0):
        return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)

    H, G, W, U = normal(T, d), normal(r, d, scale=d ** -0.5), normal(n, r, d, d, scale=d ** -0.5), normal(V, d, scale=d ** -0.5)
    X = torch.randint(0, V, (T, n), generator=gen, device="cuda", dtype=torch.int32)
    got = []
    for flags in (0, binding.MIN_WORKSPACE):
        ds = binding.make_desc(T, d, V, n, r, binding.BF16, flags)
        ctx = torch.empty(binding.cp_head_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
        ws = torch.empty(max(binding.cp_head_workspace_bytes(ds, op) for op in (binding.OP_LOSS_FWD, binding.OP_LOSS_BWD)),
                         dtype=torch.uint8, device="cuda")
        out = [torch.empty(s, dtype=torch.float32, device="cuda") for s in ((T,), (T, d), (n, r, d, d), (V, d), (r, d))]
        binding.cp_head_loss_fwd(ds, H, W, U, G, X, out[0], ctx, ws)
        binding.cp_head_loss_bwd(ds, H, W, U, G, X, None, 1.0 / T, ctx, *out[1:], ws)
        torch.cuda.synchronize()
        got.append(out)
    assert torch.equal(got[0][0], got[1][0])
    dU = [out[3] for out in got]
    # the same products of bf16; K = 131200 roundings of a running sum, each by at most 2^-25 of it, drift like a random walk:
    # sqrt(K) 2^-25 = 1.1e-5 for either order.  Row by row as well, so that a misplaced tile is not lost in the norm.
    assert (dU[0] - dU[1]).norm() <= 2e-5 * dU[1].norm()
    assert ((dU[0] - dU[1]).norm(dim=1) <= 1e-4 * dU[1].norm(dim=1)).all()


@pytest.mark.parametrize("shape", FULL_HEADS, ids=lambda s: "x".join(map(str, s)))
def test_full_heads(oracle, shape):
    import torch
    from paper_2410_17765_amd import binding, head
    T, d, V, n, r = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(7)
    H, F, G = (synth.bf16_round(rng.standard_normal(s).astype(np.float32) * c)
               for s, c in (((T, d), 1), ((n, r, V, d), d ** -0.5), ((r, d), d ** -0.5)))
    X = rng.integers(0, V, (T, n), dtype=np.int32)
    X[::7, n - 1] = -1
    ref = oracle.full_loss_bwd(H, F, G, X)
    Hd, Xd = head.to_device(H, "bf16"), torch.from_numpy(X).cuda()
    got = {}
    for flags in (0, binding.MIN_WORKSPACE):
        h = head.CpFullHead(F, G, dtype="bf16", flags=flags)
        h.loss_fwd(Hd, Xd)
        got[flags] = {k: v.cpu().numpy() for k, v in h.loss_bwd(Hd, Xd).items()}
        for k, v in ref.items():
            assert rel_fro(got[flags][k], v) <= 1e-2, (flags, k)
    # dz is the same; fp32 sums of up to 1500 terms in another order
    for k in ref:
        assert rel_fro(got[0][k], got[binding.MIN_WORKSPACE][k]) <= 1e-5, k
