"""A new batch plan picks its launch form by the number of matrices and takes its tiles in 64 x 64 pieces
where that is less work: bitwise the results of both explicit tiles and both launch forms, at sizes
around the tiles, the row chunks of the bounds pass (16 rows) and the paddings. A matrix with a
non-finite element fails by itself."""
import pytest

from paper_2605_08523_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 257]


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("count,form", [(11, "layers"), (12, "queue")])
def test_default_plan_equals_explicit_ones(api, paper_model, count, form, prec):
    print(f"case count={count} {prec}", flush=True)
    mats = [dict(H=torch.from_numpy(W.random_dense(n, 400 + n)).cuda(), mu=0.02, kT=0.1)
            for n in SIZES[:count]]
    mats[5]["H"][3, 3] = float("inf")
    plan = api.BatchPlan(mats, paper_model, prec=prec)
    assert plan.launch_form == form and plan.tile == 128
    plan.launch()
    torch.cuda.synchronize()
    D, tr, status = [d.clone() for d in plan.D], plan.tr.clone(), plan.status.clone()
    assert status[5].item() == api.FE_ERR_NONFINITE and torch.isnan(tr[5]).all()
    for tile in (128, 64):
        if tile == 64 and prec == "bf16x3":
            continue
        plan.retile(tile)
        for launch in ("layers", "queue"):
            plan.set_launch(launch)
            for _ in range(3):
                plan.launch()
            torch.cuda.synchronize()
            for b in range(count):
                if b != 5:
                    assert torch.equal(plan.D[b], D[b]), (tile, launch, SIZES[b])
            assert torch.equal(plan.status, status)
    plan.close()


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("count", [28, 30])
def test_batches_about_the_staged_line(api, paper_model, count, prec):
    # 63.0 and 67.5 MiB of operands: just below and above the line of the register-staged launches
    print(f"case staged count={count} {prec}", flush=True)
    ns = [(765, 768, 700, 641)[b % 4] for b in range(count)]
    mats = [dict(H=torch.from_numpy(W.random_dense(n, 600 + b)).cuda(), mu=0.02, kT=0.1)
            for b, n in enumerate(ns)]
    mats[7]["H"][600, 3] = float("nan")
    ref = []
    for m in mats[:4]:
        plan = api.BatchPlan([m], paper_model, prec=prec)   # one matrix: never staged
        plan.launch()
        torch.cuda.synchronize()
        ref.append(plan.D[0].clone())
        plan.close()
    plan = api.BatchPlan(mats, paper_model, prec=prec)
    plan.retile(128)
    first = None
    for launch in ("layers", "queue"):
        plan.set_launch(launch)
        for _ in range(3):
            plan.launch()
        torch.cuda.synchronize()
        assert [int(s) for s in plan.status] == [api.FE_ERR_NONFINITE if b == 7 else 0 for b in range(count)]
        for b, d in enumerate(ref):
            assert torch.equal(plan.D[b], d), (launch, b)
        if first is None:
            first = [d.clone() for d in plan.D]
        assert all(torch.equal(x, y) for b, (x, y) in enumerate(zip(first, plan.D)) if b != 7), launch
    plan.close()
