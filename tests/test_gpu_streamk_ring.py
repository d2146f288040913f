"""Stream-K over 128 x 128 ring tiles (two-part splits, n > 2816) at the edges of its range: just past
the one-round tiles (276 tiles on 256 compute units), with whole-tile rounds first (n = 4200), and where
the 256 x 256 tiles take over and hand back. Sums of 512 products added in a fixed order, so D is no
further off FP64 than the batch kernel's one chain per element, and the same on every call."""
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
@pytest.mark.parametrize("n", [2817, 2944, 4200, 4864, 4865, 5632, 5633])
def test_no_further_off_than_one_chain(api, paper_model, monkeypatch, n, prec):
    monkeypatch.delenv("FE_SCHEDULE", raising=False)
    print(f"case n={n} {prec}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    H = (H + H.T) / (2.0 * n ** 0.5)
    ws = api.Workspace(n)
    assert api.autotune_lookup(n, prec=prec, ws=ws) == ("sk256" if n in (4865, 5632) else "sk2x128")
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
    assert torch.equal(D, D.T) and e[0] <= e[1]
    # the traces are those of D before its rounding to FP32: n elements of at most 1
    assert abs(tr.item() - D.double().trace().item()) <= n * 2.0 ** -24
    ws.close()
