"""bench.py quotes a committed profile figure only for the layer kernel that the run's schedule takes:
the records of another schedule or precision, or of other sources, are not reported for it (CPU only)."""
import hashlib
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_records_follow_the_kernel(tmp_path, monkeypatch):
    h = hashlib.sha256()
    for f in bench.KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2605_08523_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    path = tmp_path / "counters.md"
    recs = [dict(kernel="k_layer_sk<fp16,128>", source_sha256="0", bytes_per_launch=1.0),
            dict(kernel="k_layer_sk<fp16,128>", source_sha256=h.hexdigest(), bytes_per_launch=2.0),
            dict(kernel="k_layer_sk<fp16,256>", source_sha256=h.hexdigest(), bytes_per_launch=3.0)]
    path.write_text("# counters\n\n" + "".join(f"traffic_json: {json.dumps(r)}\n" for r in recs))
    monkeypatch.setattr(bench, "COUNTER_SUMMARY", str(path))
    got = {s: bench.measured_traffic(bench.layer_kernel(s, "fp16x2")) for s in ("sk2x128", "sk256", "dp128")}
    assert got == {"sk2x128": 2.0, "sk256": 3.0, "dp128": None}
    assert bench.measured_traffic(bench.layer_kernel("sk2x128", "bf16x2")) is None
    path.write_text("no record\n")
    assert bench.measured_traffic("k_layer_sk<fp16,128>") is None
