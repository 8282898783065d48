"""The traffic figures of bench.py belong to the code they were counted on."""
import json

import bench


def test_each_part_of_a_kernel_has_a_definition_of_its_own(tmp_path, monkeypatch):
    names = ["k_rep_chase", *bench.KERNEL_PARTS]
    shas = [bench.kernel_source_sha(bench.KERNEL_PARTS.get(n, n)) for n in names]
    assert all(shas) and len(set(shas)) == len(names)
    # counters taken on one part's code are reported for that part only
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "kernel_source_sha", lambda k: "sha of " + k)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    for n, sha in (("k_key_edges (orphans)", "sha of orphan_scan"), ("k_key_edges (store)", "sha of orphan_scan")):
        c = {"kernel": n, "workload": "w", "kernel_sha256_16": sha, "traffic_bytes_per_launch": 7}
        (tmp_path / "profiles" / f"{n[12:-1]}.counters.json").write_text(json.dumps(c))
    assert bench.measured_traffic("k_key_edges (orphans)", "w") == 7
    assert bench.measured_traffic("k_key_edges (store)", "w") is None
