"""FE_SCHEDULE names a schedule exactly: sk256 (as the tuner prints it) and sk are the 256 x 256 tiles, only
sk2 and sk2-handover the 128 x 128 ones."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("name,schedule", [("dp", "dp128"), ("dp128", "dp128"), ("sk", "sk256"), ("sk256", "sk256"),
                                           ("sk2", "sk2x128"), ("sk2-handover", "sk2x128")])
def test_schedule_of_a_name(monkeypatch, name, schedule):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    print(f"case {name}", flush=True)
    ws = api.Workspace(1536)   # with stream-K buffers
    monkeypatch.setenv("FE_SCHEDULE", name)
    assert api.autotune_lookup(1536, prec="fp16x2", ws=ws) == schedule
    ws.close()
