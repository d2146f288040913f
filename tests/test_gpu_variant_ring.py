"""The variants' squarings on the operand ring (64 x 64 tiles for padded sizes up to 1920, 128 x 128 up
to 2816, on 256 compute units), at the edges of those ranges, bitwise against the register-staged tiles
of larger matrices: H bordered to n = 2880 by a diagonal inside its spectrum has the same bounds, and
every element of D takes the same products followed by exact zeros."""
import pytest

from paper_2605_08523_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def var():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api, variants
    api.lib()
    return variants


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [2, 64, 129, 1920, 1921, 2816])
def test_bitwise_equal_to_the_staged_tiles(var, paper_model, n, prec):
    print(f"case n={n} {prec}", flush=True)
    H = torch.from_numpy(W.random_dense(n, n)).cuda()
    mu = float(H.diagonal().mean())
    big = torch.diag(torch.full((2880,), mu, dtype=torch.float64, device="cuda"))
    big[:n, :n] = H
    q = var.embed_mlsp2(paper_model, "skip")
    D = var.expand_density_variant(H, mu, 0.1, q, prec=prec)[0]
    Db = var.expand_density_variant(big, mu, 0.1, q, prec=prec)[0]
    torch.cuda.synchronize()
    assert torch.equal(D, Db[:n, :n]) and torch.equal(D, D.T)
    assert torch.count_nonzero(Db[:n, n:]).item() == 0
