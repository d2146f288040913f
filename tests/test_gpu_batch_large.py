"""A batch matrix of 4 GiB in FP32 (padded size 32768): its 64 x 64 tiles address the state,
the accumulator and the operands beyond 32 bits, and D is bitwise that of the 128 x 128 tiles, whose
staged kernel forms 64-bit addresses. Two layers: one that writes the next state, and the last."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_tiles_beyond_4_gib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    n = 32641
    print(f"case n={n}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    H = torch.rand((n, n), dtype=torch.float64, device="cuda", generator=g)
    H -= 0.5
    H = H + H.T
    m = api.make_model([[1.0, 0.0, 0.0, 0.25], [-1.0, 2.0, 0.0, -0.5]], 40.0, 0.5)
    plan = api.BatchPlan([dict(H=H, mu=0.0, kT=1e3)], m)
    plan.set_launch("layers")
    plan.retile(128)
    plan.launch()
    torch.cuda.synchronize()
    print("128 x 128 tiles done", flush=True)
    want = plan.D[0].clone()
    plan.D[0].fill_(float("nan"))
    plan.retile(64)
    plan.launch()
    torch.cuda.synchronize()
    assert plan.status.tolist() == [0]
    assert torch.equal(plan.D[0], want)
    assert torch.count_nonzero(want[-1]).item() > n // 2
    plan.close()
