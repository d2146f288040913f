"""Stream-K over 128 x 128 tiles (two-part splits, n > 1920) at the edges of its forms: a workgroup per
ring tile that sums the plan's segments itself (n <= 2816 on 256 compute units), and the plan with
hand-overs beyond, with whole-tile rounds first at n = 5700. Segments are added in a fixed order, so D
is the same on every call, within the expansion's accuracy bar of FP64, and for FP16x2 no further off
than one chain."""
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


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [1921, 2048, 2816, 2817, 2944, 4200, 5700])
def test_no_further_off_than_one_chain(api, paper_model, monkeypatch, n, prec):
    monkeypatch.delenv("FE_SCHEDULE", raising=False)
    print(f"case n={n} {prec}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    H = (H + H.T) / (2.0 * n ** 0.5)
    ws = api.Workspace(n)
    assert api.autotune_lookup(n, prec=prec, ws=ws) == "sk2x128"
    D, tr, tr2, _ = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=ws)
    for _ in range(3):
        again, tr_a, tr2_a, _ = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=ws)
        assert torch.equal(D, again) and tr.item() == tr_a.item() and tr2.item() == tr2_a.item()
    f, v = torch.linalg.eigh(H)
    ref = (v * torch.sigmoid((0.05 - f) / 0.1)) @ v.T
    del v
    monkeypatch.setenv("FE_SCHEDULE", "dp")
    chain = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=ws)[0]
    e = [float(torch.linalg.norm(x.double() - ref)) for x in (D, chain)]
    print(f"n={n} {prec} |dD|_F {e[0]:.3e} one chain {e[1]:.3e}", flush=True)
    assert torch.equal(D, D.T) and e[0] <= 1e-5 * n
    if prec == "fp16x2":   # the sums' rounding shows; BF16x2's error is that of its 16-bit operands
        assert e[0] <= e[1]
    # the traces are those of D before its rounding to FP32: n elements of at most 1
    assert abs(tr.item() - D.double().trace().item()) <= n * 2.0 ** -24
    ws.close()
