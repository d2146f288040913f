"""Two-part layers whose 128 x 128 tiles all run at once: the kernel that sums the plan's segments by
itself gives bit for bit what the plan's workgroups give that publish partial tiles and wait for them
(FE_SCHEDULE=sk2-handover), from one tile to the last size of one round on 256 compute units."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [100, 300, 1000, 1921, 2049, 2816])
def test_segments_equal_handed_over_partials(paper_model, monkeypatch, n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    print(f"case n={n} {prec}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    H = (H + H.T) / (2.0 * n ** 0.5)
    ws = api.Workspace(max(n, 1536))   # with stream-K buffers
    out = {}
    for form in ("sk2", "sk2-handover"):
        monkeypatch.setenv("FE_SCHEDULE", form)
        assert api.autotune_lookup(n, prec=prec, ws=ws) == "sk2x128"
        D, tr, tr2, info = api.expand_density(H, 0.05, 0.1, paper_model, prec=prec, ws=ws, want_info=True)
        assert info["rc"] == 0
        out[form] = (D, tr.item(), tr2.item())
    a, b = out["sk2"], out["sk2-handover"]
    assert torch.equal(a[0], b[0])
    # the same FP64 terms, summed over the tile by eight or by four waves
    tol = 2.0 ** -53 * n * n
    assert abs(a[1] - b[1]) <= tol * n and abs(a[2] - b[2]) <= tol * n
    ws.close()
