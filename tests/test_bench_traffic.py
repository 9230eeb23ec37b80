"""The committed HBM traffic of the CG iteration kernel that bench.py reports."""
import json

import bench


def test_iteration_kernel_traffic(tmp_path, monkeypatch):
    F = 8 * 512 * 512 * 16
    with open(bench.TRAFFIC_FILE) as f:
        t = json.load(f)
    assert t["kernel"].startswith("k_cg_step") and t["field_bytes"] == F
    # at least the algorithmic bytes (4F, and 7F where x is updated), at most
    # those plus two cells of halo per tile of four rows, of r and p
    odd, even = t["by_parity"]["odd_k"], t["by_parity"]["even_k"]
    assert 4 * F <= odd <= 5.2 * F and 7 * F <= even <= 8.2 * F
    mean = bench.measured_traffic(F, 4)
    if t["kernel_source_sha256_16"] == bench.kernel_source_hash():
        assert mean == bench.measured_traffic(F, 16) and 5.5 * F <= mean <= 6.7 * F
    else:
        assert mean is None
    assert bench.measured_traffic(2 * F, 4) is None
    fresh = dict(t, kernel_source_sha256_16=bench.kernel_source_hash())
    p = tmp_path / "traffic.json"
    p.write_text(json.dumps(fresh))
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(p))
    assert bench.measured_traffic(F, 4) == sum(t["by_parity"].values()) / 2
