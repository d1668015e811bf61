"""Log-normalisers of the teacher's rows on both sides of each line between the forms that compute them (512, 8192 columns; what each
holds in registers between the maximum and the sum: 8192 and 32768; their chunks of 2048 and 4096), against float64.  With beta = 1
and a head whose every distribution is uniform the loss is log V - H(p^c), which takes them and nothing else that rounds much."""
import pytest

pytestmark = pytest.mark.gpu

VOCABULARIES = [1, 255, 512, 513, 2049, 4095, 8192, 8193, 12289, 32768, 32777, 70001]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", VOCABULARIES)
def test_entropy_of_the_teacher(V, dtype):
    import torch
    from paper_2410_17765_amd import binding
    T, d, n, r = 5, 64, 1, 2
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    H = torch.randn(T, d, generator=gen, device="cuda").to(store)
    G, W, U = torch.zeros(r, d, dtype=store, device="cuda"), torch.zeros(n, r, d, d, dtype=store, device="cuda"), torch.zeros(V, d, dtype=store, device="cuda")
    TZ = (torch.randn(T, n, V, generator=gen, device="cuda") * 2.0).to(store)
    X = torch.zeros(T, n, dtype=torch.int32, device="cuda")
    ds = binding.make_desc(T, d, V, n, r, binding.BF16 if dtype == "bf16" else binding.FP32, 0)
    ctx = torch.zeros(binding.cp_head_distill_ctx_bytes(ds), dtype=torch.uint8, device="cuda")
    ws = torch.full((binding.cp_head_workspace_bytes(ds, binding.OP_DISTILL_FWD),), 255, dtype=torch.uint8, device="cuda")
    loss = torch.empty(T, device="cuda")
    binding.cp_head_distill_loss_fwd(ds, H, W, U, G, X, TZ, 1.0, 1.0, loss, ctx, ws)
    logp = torch.log_softmax(TZ[:, 0].double(), dim=1)
    expected = torch.log(torch.tensor(float(V), dtype=torch.float64)).item() + (logp.exp() * logp).sum(dim=1)
    # KL is a sum of V terms p (log p + log V) of at most log V + 12 each, weighted by probabilities with relative errors of 2^-20
    assert (loss.double() - expected).abs().max() <= 2.0 ** -20 * 4 * (12 + expected.abs().max())
