"""Small matrices with all layers in one launch (n <= 448 for the 16-bit splits, n <= 192 for FP32 and
FP64 on 256 compute units; from the bounds to the traces in one workgroup for n <= 64 in FP64 and 80 in
FP32), at the edges of their tiles and of the sizes they are chosen for. The
splits take the tile code of the launches per layer, so D is bitwise that of a batch of one, call
after call; FP32 and FP64 are held to the oracle's recursion by the rounding of their chains of n
products over 26 layers. A wait that gives up is reported as for stream-K."""
import numpy as np
import pytest

from oracle import fermi as F
from oracle import recursion as R
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


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("fp64", 1e-11)])
@pytest.mark.parametrize("n", [1, 16, 17, 48, 64, 65, 80, 81, 128, 129, 192, 193])
def test_wide_against_the_oracle(api, paper_model, n, prec, tol):
    print(f"case n={n} {prec}", flush=True)
    Hh = W.random_dense(n, 90 + n)
    H = torch.from_numpy(Hh).cuda()
    m = paper_model
    ref, _ = R.mlsp2_density(Hh, 0.05, 0.1, m.theta, m.beta0, m.mu0)
    ws = api.Workspace(n)
    out = torch.float64 if prec == "fp64" else torch.float32
    first = None
    for _ in range(10):
        D, tr, tr2, info = api.expand_density(H, 0.05, 0.1, m, prec=prec, ws=ws, out_dtype=out,
                                              want_info=True)
        torch.cuda.synchronize()
        first = D.clone() if first is None else first
        assert torch.equal(D, first) and torch.equal(D, D.T)
    lo, hi = F.gershgorin(Hh)
    assert abs(info["emin"] - lo) <= 1e-14 * n and abs(info["emax"] - hi) <= 1e-14 * n
    d = D.double().cpu().numpy()
    assert np.linalg.norm(d - ref) / max(1.0, np.linalg.norm(ref)) <= tol
    # D's elements leave in its type, the trace is summed from the FP64 / FP32 layer values
    assert abs(float(tr) - np.trace(ref)) <= tol * n
    assert abs(float(tr2) - np.sum(ref * ref)) <= 2 * tol * n
    ws.close()


@pytest.mark.parametrize("n,prec", [(128, "fp16x2"), (128, "fp64")])
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


@pytest.mark.parametrize("n,prec", [(50, "fp64"), (70, "fp32"), (150, "fp64"), (300, "fp16x2"), (600, "bf16x2")])
def test_captured_replays_equal_the_eager_call(api, paper_model, n, prec):
    print(f"case capture n={n} {prec}", flush=True)
    H = torch.from_numpy(W.random_dense(n, 17)).cuda()
    out = torch.float64 if prec == "fp64" else torch.float32
    want, tr, tr2, _ = api.expand_density_noalloc(H, 0.05, 0.1, paper_model, prec=prec, out_dtype=out)
    want, tr = want.clone(), tr.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        D, trc, _, _ = api.expand_density_noalloc(H, 0.05, 0.1, paper_model, prec=prec, out_dtype=out)
    for _ in range(4):
        D.zero_()
        other = api.expand_density(H, 0.0, 0.1, paper_model, prec=prec, ws=api.workspace(n))[0]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(D, want) and trc.item() == tr.item() and not torch.equal(other, want)
