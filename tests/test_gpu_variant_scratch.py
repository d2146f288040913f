"""The caller's scratch of a Skip-SP2 / Max-SP2 expansion may start on any float: from 4 bytes past a
16-byte boundary (register-staged tiles) D and the traces are those of an aligned scratch (ring tiles,
64 x 64 and 128 x 128, squarings fused with the next combine)."""
import pytest

from paper_2605_08523_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("arch", ["skip", "max"])
@pytest.mark.parametrize("n,prec", [(130, "fp16x2"), (1000, "bf16x2"), (2100, "fp16x2")])
def test_scratch_on_any_float(paper_model, n, prec, arch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import variants
    print(f"case n={n} {prec} {arch}", flush=True)
    H = torch.from_numpy(W.random_dense(n, n)).cuda()
    q = variants.embed_mlsp2(paper_model, arch)
    nbytes = variants.scratch_bytes(n, q)
    out = []
    for off in (0, 4):
        scratch = torch.empty(nbytes + 16, dtype=torch.uint8, device="cuda")[off:off + nbytes]
        assert scratch.data_ptr() % 16 == off
        D, tr, tr2, _ = variants.expand_density_variant(H, 0.02, 0.1, q, prec=prec, scratch=scratch)
        torch.cuda.synchronize()
        out.append((D, tr.item(), tr2.item()))
    assert torch.equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
