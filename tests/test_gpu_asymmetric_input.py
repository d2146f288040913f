"""H that is not exactly symmetric: an element of D takes H's element above the diagonal as the state
of the first layer, and whole rows of H in its product; from the second layer on everything is
symmetric, so D is exactly symmetric too. The lower triangle is perturbed by 1e-2, far above the
tolerance (the accuracy bar of the expansion), so a layer that used the wrong element would show."""
import numpy as np
import pytest

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


def reference(H, mu, kT, m):
    X, info = R.rescale(H, mu, kT, m.beta0, m.mu0)
    state = np.triu(X) + np.triu(X, 1).T
    acc = np.zeros_like(X)
    for a, b, c, d in np.asarray(m.theta).reshape(-1, 4):
        acc += d * state
        X = state = a * (X @ X.T) + b * state + c * np.eye(len(H))
    D = acc + state
    return np.eye(len(H)) - D if info["flipped"] else D


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3", "fp32", "fp64"])
@pytest.mark.parametrize("n", [50, 100, 150, 500, 2000])
def test_state_comes_from_above_the_diagonal(api, paper_model, n, prec):
    print(f"case n={n} {prec}", flush=True)
    m = paper_model
    H = W.random_dense(n, 300 + n)
    g = np.random.default_rng(n)
    H = H + np.tril(1e-2 / np.sqrt(n) * g.standard_normal((n, n)), -1)
    ref = reference(H, 0.05, 0.1, m)
    Hd = torch.from_numpy(H).cuda()
    D = api.expand_density(Hd, 0.05, 0.1, m, prec=prec, ws=api.Workspace(n))[0]
    torch.cuda.synchronize()
    assert torch.equal(D, D.T)
    assert np.linalg.norm(D.double().cpu().numpy() - ref) / n <= 1e-5
    if prec in ("fp16x2", "bf16x3") and n <= 500:
        plan = api.BatchPlan([dict(H=Hd, mu=0.05, kT=0.1)], m, prec=prec)
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(plan.D[0], D)
        plan.close()
