"""A tuned schedule serves the sizes near it whose tiles run in the same form, not those across a line
where the schedules stand for other kernels (256 compute units: 64 x 64 tiles up to n = 1984, 128 x 128
in one round up to 2816, several rounds beyond)."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,near,across", [(2816, 2048, (2817, 2900, 1984)), (1984, 1500, (1985, 2500)),
                                           (2900, 2817, (2816, 2100))])
def test_tuned_entry_stays_on_its_side(n, near, across):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    ws = api.Workspace(2944)
    api.autotune_clear()
    default = {k: api.autotune_lookup(k, ws=ws) for k in across}
    try:
        r = api.autotune([n], ws=ws)[0]
        print(f"case n={n} -> {r['schedule']} {r['ms']}", flush=True)
        assert api.autotune_lookup(n, ws=ws) == api.autotune_lookup(near, ws=ws) == r["schedule"]
        assert {k: api.autotune_lookup(k, ws=ws) for k in across} == default
    finally:
        api.autotune_clear()
        ws.close()
