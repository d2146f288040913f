"""Which tile the layer kernel of a batch plan runs: 64 x 64 pieces by size on both sides of its lines,
the same whichever launch form is set, what retile asked for afterwards, and what the tuner chose. A three-part BF16 plan's tuner times the
pieces too, so tuning cannot lose the faster form that a new plan starts with (30 matrices of one or two
tiles: 1.3 times as fast); the result is the same."""
import ctypes

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


def batch(ns):
    return [dict(H=torch.from_numpy(W.random_dense(n, 10 * n + b)).cuda(), mu=0.02, kT=0.1)
            for b, n in enumerate(ns)]


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
@pytest.mark.parametrize("n,count,form,tile", [(64, 2, "layers", 64), (640, 2, "layers", 64), (641, 2, "layers", 128),
                                               (500, 9, "layers", 128), (500, 13, "queue", 64),
                                               (500, 40, "queue", 128)])
def test_tile_by_size(api, paper_model, n, count, form, tile, prec):
    print(f"case n={n} count={count} {prec}", flush=True)
    plan = api.BatchPlan(batch([n] * count), paper_model, prec=prec)
    assert plan.launch_form == form
    assert api.batch_default_tile([n] * count, paper_model.L, form, prec) == tile
    for other in (form, "layers", "queue"):
        assert plan.tile == 128 and plan.kernel_tile == tile
        plan.set_launch(other)
    plan.retile(128)
    assert plan.tile == 128 and plan.kernel_tile == 128
    if prec == "fp16x2":
        plan.retile(64)
        assert plan.tile == 64 and plan.kernel_tile == 64
    plan.close()


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
def test_tuning_times_the_form_of_a_new_plan(api, paper_model, prec):
    print(f"case autotune {prec}", flush=True)
    plan = api.BatchPlan(batch([64 + 4 * b for b in range(30)]), paper_model, prec=prec)
    assert plan.kernel_tile == 64
    plan.launch()
    torch.cuda.synchronize()
    want = [d.clone() for d in plan.D]
    tile, ms = plan.autotune()
    assert tile == plan.tile == (64 if prec == "fp16x2" else 128) and plan.kernel_tile == 64
    assert set(ms) == ({64, 128} if prec == "fp16x2" else {128})
    plan.launch()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(plan.D, want))
    plan.close()


def test_argument_errors(api):
    tile = ctypes.c_int32()
    assert api.lib().fe_batch_plan_kernel_tile(None, ctypes.byref(tile)) == api.FE_ERR_ARG
