"""Small matrices with all layers in one launch (n <= 448 for the 16-bit splits on 256 compute
units), at the edges of their tiles and of the sizes they are chosen for. They take the tile code of
the launches per layer, so D is bitwise that of a batch of one, call after call. A
wait that gives up is reported as for stream-K."""
import pytest

from paper_2605_08523_amd import workloads as W

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
@pytest.mark.parametrize("n", [1, 64, 65, 447, 448, 449])
def test_split_bitwise_and_repeatable(api, paper_model, n, prec):
    print(f"case n={n} {prec}", flush=True)
    H = torch.from_numpy(W.random_dense(n, 70 + n)).cuda()
    ws = api.Workspace(n)
    plan = api.BatchPlan([dict(H=H, mu=0.05, kT=0.1)], paper_model, prec=prec)
    plan.launch()
    for _ in range(10):
        D = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=ws)[0]
        torch.cuda.synchronize()
        assert torch.equal(D, plan.D[0]) and torch.equal(D, D.T)
    plan.close()
    ws.close()


@pytest.mark.parametrize("n,prec", [(128, "fp16x2")])
def test_giveup_is_reported(api, paper_model, n, prec):
    print(f"case giveup n={n} {prec}", flush=True)
    H = torch.from_numpy(W.random_dense(n, 5)).cuda()
    ws = api.Workspace(n)
    good = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws)[0]
    api.debug_streamk_giveup(True)
    try:
        D, tr, tr2, _ = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws)
        torch.cuda.synchronize()
        assert torch.isnan(tr).item() and torch.isnan(tr2).item() and torch.isnan(D).any().item()
        with pytest.raises(api.FeError) as e:
            api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws, want_info=True)
        assert e.value.code == api.FE_ERR_HIP
    finally:
        api.debug_streamk_giveup(False)
    D, _, _, info = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws, want_info=True)
    assert info["rc"] == 0 and torch.equal(D, good)
    ws.close()
