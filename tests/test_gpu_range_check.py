"""The 16-bit modes refuse a model whose operands leave [-16, 16] on the unit interval of its input. The
largest value sits at the first, the last or the middle sample point, exactly at the bound (accepted)
and one part in 2^40 beyond it (refused)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BEYOND = 16.0 * (1.0 + 2.0 ** -40)


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api as _api
    _api.lib()
    return _api


def accepted(api, call):
    try:
        call()
        return True
    except api.FeError as e:
        assert e.code == api.FE_ERR_RANGE
        return False


@pytest.mark.parametrize("top,ok", [(16.0, True), (BEYOND, False)])
@pytest.mark.parametrize("where", ["first", "last", "middle", "later layer"])
def test_layer_range(api, where, top, ok):
    # x' = a x^2 + b x + c with |x'| = top at the named input and smaller elsewhere
    theta = {"first": [[0.0, -top, top, 0.0]], "last": [[0.0, -top, 0.0, 0.0]],
             "middle": [[-4.0 * top, 4.0 * top, 0.0, 0.0]],
             "later layer": [[0.0, 1.0, 0.0, 0.5], [0.0, top, 0.0, 0.0]]}[where]
    m = api.make_model(np.array(theta), 100.0, 1.0 / 3.0)
    H = torch.diag(torch.linspace(-1.0, 1.0, 40, dtype=torch.float64, device="cuda"))
    ws = api.Workspace(40)
    assert accepted(api, lambda: api.expand_density(H, 0.0, 0.1, m, prec="fp16x2", ws=ws)) is ok
    ws.close()


@pytest.mark.parametrize("top,ok", [(16.0, True), (BEYOND, False)])
@pytest.mark.parametrize("arch", ["max", "skip"])
@pytest.mark.parametrize("where", ["first", "last"])
def test_variant_range(api, arch, where, top, ok):
    from paper_2605_08523_amd import variants
    c0, c1 = (top, -top) if where == "first" else (0.0, top)
    # one layer z = c0 + c1 x, then an output that uses z^2 alone
    coef = [c0, c1, 0.0, 0.0, 1.0] if arch == "max" else [c0, c1, 0.0, 0.0, 0.0, 1.0]
    q = variants.QModel(arch, 1, np.array(coef), 100.0, 1.0 / 3.0, 1, 1)
    H = torch.diag(torch.linspace(-1.0, 1.0, 40, dtype=torch.float64, device="cuda"))
    assert accepted(api, lambda: variants.expand_density_variant(H, 0.0, 0.1, q)) is ok
