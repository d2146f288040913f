"""A wait that gives up inside a launch over several layers must not let the next layer start on operands
that a late workgroup has yet to store: the item is not counted, so the layers after it give up as well
and come out as NaN. One tile of the last layer but one gives up here; the last layer's tiles away from
its row and column hold none of its NaN unless their own waits give up."""
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


@pytest.mark.parametrize("n,prec,tiles", [(256, "fp16x2", 10), (256, "bf16x3", 10), (128, "fp64", 10),
                                          (160, "fp32", 21)])
def test_resident_layers_after_a_giveup(api, paper_model, n, prec, tiles):
    print(f"case n={n} {prec}", flush=True)
    H = torch.from_numpy(W.random_dense(n, 7)).cuda()
    ws = api.Workspace(n)
    good = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws)[0].clone()
    api.debug_resident_giveup((paper_model.L - 2) * tiles)
    try:
        D, tr, tr2, _ = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws)
        torch.cuda.synchronize()
        assert torch.isnan(D).all().item() and torch.isnan(tr).item() and torch.isnan(tr2).item()
        with pytest.raises(api.FeError) as e:
            api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws, want_info=True)
        assert e.value.code == api.FE_ERR_HIP
    finally:
        api.debug_resident_giveup(-1)
    D, _, _, info = api.expand_density(H, 0.1, 0.1, paper_model, prec=prec, ws=ws, want_info=True)
    assert info["rc"] == 0 and torch.equal(D, good)
    ws.close()


@pytest.mark.parametrize("ns,tile,prec", [((300, 130, 520), 64, "fp16x2"), ((300, 130, 520), 128, "fp16x2"),
                                          ((300, 130, 520), 128, "bf16x3"), ((768,) * 30, 128, "fp16x2"),
                                          ((768,) * 30, 128, "bf16x3")])
def test_batch_layers_after_a_giveup(api, paper_model, ns, tile, prec):
    print(f"case {len(ns)} matrices tile={tile} {prec}", flush=True)   # 30: the staged launch
    mats = [dict(H=torch.from_numpy(W.random_dense(n, n + b)).cuda(), mu=0.02, kT=0.1)
            for b, n in enumerate(ns)]
    plan = api.BatchPlan(mats, paper_model, prec=prec)
    api.debug_batch_queue_giveup_layer(paper_model.L - 2)
    try:
        plan.set_launch("queue")
        plan.retile(tile)
    finally:
        api.debug_batch_queue_giveup_layer(-1)
    plan.launch()
    torch.cuda.synchronize()
    assert plan.status.tolist() == [api.FE_ERR_HIP] * len(ns) and torch.isnan(plan.tr).all().item()
    assert all(torch.isnan(d).all().item() for d in plan.D)
    plan.retile(tile)
    plan.launch()
    torch.cuda.synchronize()
    assert plan.status.tolist() == [0] * len(ns) and not any(torch.isnan(d).any().item() for d in plan.D)
    plan.close()
