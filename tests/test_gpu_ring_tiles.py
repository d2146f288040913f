"""One-round data-parallel layers (64 x 64 and 128 x 128 tiles, direct-to-LDS operand ring) at the
edges of their tiles and of the sizes they are chosen for (n <= 1984 and n <= 2816 on 256 compute
units): they take the same products in the same order as a batch of one, whose launch form and tile
are other ones, or the same ring tiles in another launch (the register-staged kernel is the partner at
n = 2817 alone), so D is bitwise the batch's. The traces are FP64 sums of the same values in
another order: n^2 additions of at most 1 each, 2^-53 relative each."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 191, 449, 1983, 1985, 2816, 2817])
def test_bitwise_equal_to_the_batch_kernel(api, paper_model, monkeypatch, n, prec):
    monkeypatch.setenv("FE_SCHEDULE", "dp")   # n = 2817 takes the kernel of more rounds
    print(f"case n={n} {prec}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    H = (H + H.T) / (2.0 * n ** 0.5)
    D, tr, tr2, _ = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=api.Workspace(n + 1))
    plan = api.BatchPlan([dict(H=H, mu=0.05, kT=0.1)], paper_model, prec=prec)
    plan.launch()
    torch.cuda.synchronize()
    assert torch.equal(D, plan.D[0])
    tol = 2.0 ** -53 * n * n
    assert abs(float(tr) - float(plan.tr[0, 0])) <= tol * n
    assert abs(float(tr2) - float(plan.tr[0, 1])) <= tol * n
    plan.close()
