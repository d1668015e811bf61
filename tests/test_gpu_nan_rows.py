"""A NaN in the unembedding reaches every result of the matrix-core path that its logits belong to, also where the damaged rows are all
that a segment of the row statistics holds (the last rows of a vocabulary one or two past a multiple of 128: no maximum shows them).
Every form of the z product: straight from memory for up to 16 and 32 head rows, tiles of 64 and of 256 rows."""
import pytest

pytestmark = pytest.mark.gpu


def normal(gen, *size, scale=1.0):
    import torch
    return (torch.randn(size, generator=gen, device="cuda") * scale).to(torch.bfloat16)


def setup(T, d, V, n, r, flags=0):
    import torch
    from paper_2410_17765_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    print(f"case T {T} d {d} V {V} n {n} r {r} flags {flags}", flush=True)
    U = normal(gen, V, d, scale=d ** -0.5)
    U[V // 128 * 128:] = float("nan")
    return dict(ds=binding.make_desc(T, d, V, n, r, binding.BF16, flags), H=normal(gen, T, d), G=normal(gen, r, d, scale=d ** -0.5),
                W=normal(gen, n, r, d, d, scale=d ** -0.5), U=U, X=torch.randint(0, 64, (T, n), generator=gen, device="cuda", dtype=torch.int32),
                TZ=normal(gen, T, n, V), loss=torch.zeros(T, device="cuda"), dH=torch.zeros(T, d, device="cuda"))


def scratch(size):
    import torch
    return torch.zeros(max(int(size), 256), dtype=torch.uint8, device="cuda")


# head rows (T r): 1, 16, 17, 32, 40, 64, 65, 512
@pytest.mark.parametrize("V", [129, 1025, 32001, 40322, 131073])
@pytest.mark.parametrize("T,r", [(1, 1), (2, 8), (17, 1), (4, 8), (5, 8), (64, 1), (65, 1), (64, 8)])
def test_first_token(T, r, V):
    import torch
    from paper_2410_17765_amd import binding
    s = setup(T, 64, V, 1, r)
    logp = torch.zeros(T, V, device="cuda")
    binding.cp_head_first_token_logprob(s["ds"], s["H"], s["W"], s["U"], s["G"], logp,
                                        scratch(binding.cp_head_workspace_bytes(s["ds"], binding.OP_FIRST_TOKEN)))
    assert torch.isnan(logp).all()


@pytest.mark.parametrize("T,n,r", [(1, 1, 1), (2, 1, 8), (2, 2, 8), (8, 4, 4), (40, 1, 8), (2, 2, 16)])
def test_draft_and_sequential(T, n, r):
    import torch
    from paper_2410_17765_amd import binding
    V = 1025
    s = setup(T, 64, V, n, r)
    alpha, tokens, logq = (torch.zeros(x, dtype=t, device="cuda") for x, t in ((T, torch.int32), ((T, n), torch.int32), (T, torch.float32)))
    u = torch.full((T, 1 + n), 0.5, device="cuda")
    binding.cp_head_draft_sample(s["ds"], s["H"], s["W"], s["U"], s["G"], u, alpha, tokens, logq,
                                 scratch(binding.cp_head_workspace_bytes(s["ds"], binding.OP_DRAFT)))
    assert torch.isnan(logq).all() and int(tokens.min()) >= 0 and int(tokens.max()) < V
    binding.cp_head_draft_sample_sequential(s["ds"], s["H"], s["W"], s["U"], s["G"], u[:, :n].contiguous(), tokens, logq,
                                            scratch(binding.cp_head_workspace_bytes(s["ds"], binding.OP_DRAFT_SEQUENTIAL)))
    assert torch.isnan(logq).all() and int(tokens.min()) >= 0 and int(tokens.max()) < V


@pytest.mark.parametrize("V", [129, 1026, 40001])
@pytest.mark.parametrize("kind", ["pair", "keep", "single", "full", "full keep", "tune", "tune keep", "tune least"])
def test_losses(kind, V):
    import torch
    from paper_2410_17765_amd import binding as b
    T, d, n, r = 37, 64, 2, 4
    s = setup(T, d, V, n, r, b.KEEP_LOGITS if "keep" in kind else b.MIN_WORKSPACE if "least" in kind else 0)
    ds, H, W, U, G, X, loss, dH = (s[k] for k in ("ds", "H", "W", "U", "G", "X", "loss", "dH"))
    if "full" in kind:
        F = U.expand(n, r, V, d).contiguous()
        ctx = scratch(b.cp_head_full_ctx_bytes(ds))
        ws = scratch(max(b.cp_head_workspace_bytes(ds, op) for op in (b.OP_FULL_LOSS_FWD, b.OP_FULL_LOSS_BWD)))
        b.cp_head_full_loss_fwd(ds, H, F, G, X, loss, ctx, ws)
        b.cp_head_full_loss_bwd(ds, H, F, G, X, None, 1.0, ctx, dH, None, None, ws)
    elif "tune" in kind:
        ctx = scratch(b.cp_head_distill_ctx_bytes(ds))
        ws = scratch(max(b.cp_head_workspace_bytes(ds, op) for op in (b.OP_DISTILL_FWD, b.OP_DISTILL_BWD)))
        b.cp_head_distill_loss_fwd(ds, H, W, U, G, X, s["TZ"], 0.9, 0.8, loss, ctx, ws)
        b.cp_head_distill_loss_bwd(ds, H, W, U, G, X, s["TZ"], None, 1.0, ctx, dH, None, None, None, ws)
    elif kind == "single":
        b.cp_head_loss_fwd_bwd(ds, H, W, U, G, X, None, 1.0, loss, dH, None, None, None, scratch(b.cp_head_workspace_bytes(ds, b.OP_LOSS_FWD_BWD)))
    else:
        ctx = scratch(b.cp_head_ctx_bytes(ds))
        ws = scratch(max(b.cp_head_workspace_bytes(ds, op) for op in (b.OP_LOSS_FWD, b.OP_LOSS_BWD)))
        b.cp_head_loss_fwd(ds, H, W, U, G, X, loss, ctx, ws)
        b.cp_head_loss_bwd(ds, H, W, U, G, X, None, 1.0, ctx, dH, None, None, None, ws)
    assert torch.isnan(loss).all() and torch.isnan(dH).all()
