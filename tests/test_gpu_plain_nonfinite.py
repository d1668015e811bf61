"""NaN and infinities in the statistics of the plain path: none of the forms in which the vocabulary is cut into tiles may
hide a NaN, and infinite logits weigh what they do in a running log-sum-exp."""
import numpy as np
import pytest

from paper_2410_17765_amd import synth
from tests.test_gpu_generic import run_loss

pytestmark = pytest.mark.gpu

# T, d, V, r: logit tiles of 128, 64 and 32 columns
CASES = [(800, 128, 3333, 4), (257, 333, 3001, 3), (300, 48, 515, 2)]


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2410_17765_amd import binding, head
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return head


def make(shape):
    T, d, V, r = shape
    cfg = synth.HeadConfig("nonfinite", T=T, d=d, V=V, n=1, r=r, dtype="fp32", targets="uniform")
    inp = synth.make_inputs(cfg)
    inp["X"][:] = np.arange(T, dtype=np.int32)[:, None] % 100
    print(f"case {cfg}", flush=True)
    return cfg, inp


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_damaged_block_of_the_unembedding(gpu, shape):
    """128 rows of U are NaN, whole tiles of every width, and no target lies among them: every logit row has NaN in it."""
    cfg, inp = make(shape)
    inp["U"][128:256] = np.nan
    loss, grads = run_loss(gpu, cfg, inp, synth.upstream_grad(cfg.T))
    assert np.isnan(loss).all()
    assert np.isnan(grads["dH"]).all() and np.isnan(grads["dU"][:128]).all()


@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_infinite_logits(gpu, shape):
    """One infinite weight of U: its logit is +infinity for some head rows (whose other tokens then have probability zero)
    and -infinity for the rest (where it does not count)."""
    cfg, inp = make(shape)
    inp["U"][200, 0] = np.inf
    loss, _ = run_loss(gpu, cfg, inp)
    H, W, U, G = (inp[k].astype(np.float64) for k in ("H", "W", "U", "G"))
    g = H @ G.T
    logw = g - np.log(np.exp(g - g.max(1, keepdims=True)).sum(1, keepdims=True)) - g.max(1, keepdims=True)
    a = np.empty_like(logw)
    for e in range(cfg.r):
        y = H @ W[0, e].T
        infinite = y[:, 0] > 0
        z = y @ np.delete(U, 200, 0).T                # where it is -infinity, token 200 adds nothing
        mx = z.max(1)
        lse = np.where(infinite, np.inf, mx + np.log(np.exp(z - mx[:, None]).sum(1)))
        a[:, e] = logw[:, e] + z[np.arange(cfg.T), inp["X"][:, 0]] - lse
    some = np.isfinite(a).any(1)
    assert 0.2 < some.mean() and (a == -np.inf).any()
    mx = a[some].max(1)
    expect = -(mx + np.log(np.exp(a[some] - mx[:, None]).sum(1)))
    # log-sum-exp over fp32 logits: a few units in the last place of the loss
    np.testing.assert_allclose(loss[some], expect, atol=4e-6 * max(1.0, np.abs(expect).max()), rtol=0)
    assert not np.isfinite(loss[~some]).any()
