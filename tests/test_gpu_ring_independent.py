"""The ring tiles of one-round layers (launch per layer and all layers in one launch) against the
register-staged kernel of more rounds, which shares neither their K loop nor their epilogue: H bordered to
n = 2900 by a diagonal inside its spectrum has the same bounds, and every element of D takes the same
products followed by exact zeros, so D is bitwise its block. Edges of the tiles and of the sizes that
take them: one launch to n = 448, 64 x 64 tiles to 1984, 128 x 128 to 2816 (256 compute units)."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("n", [2, 63, 65, 200, 448, 449, 1408, 1409, 1984, 1985, 2816])
def test_bitwise_equal_to_the_staged_kernel(paper_model, monkeypatch, n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    monkeypatch.setenv("FE_SCHEDULE", "dp")   # one chain per element in both
    print(f"case n={n} {prec}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    H = (H + H.T) / (2.0 * n ** 0.5)
    mu = float(H.diagonal().mean())
    big = torch.diag(torch.full((2900,), mu, dtype=torch.float64, device="cuda"))
    big[:n, :n] = H
    ws = api.Workspace(2900)
    D = api.expand_density(H, mu, 0.1, paper_model, prec=prec, ws=ws)[0]
    Db = api.expand_density(big, mu, 0.1, paper_model, prec=prec, ws=ws)[0]
    torch.cuda.synchronize()
    assert not torch.isnan(D).any().item()
    assert torch.equal(D, Db[:n, :n]) and torch.equal(D, D.T)
    assert torch.count_nonzero(Db[:n, n:]).item() == 0
    ws.close()
