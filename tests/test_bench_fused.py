"""bench.py's figures of the fused forms: no memory rate that assumes a sweep per
block, and each speedup named by what it is against."""

import bench


def test_entry_has_no_rate_per_block():
    e = bench.fused_entry(100.0, 800, 50, 20)
    assert e["ms"] == 100.0 and e["gates_per_s"] == 8000.0 and e["ms_per_block"] == 2.0
    assert e["TFLOPs"] == round(8 * 32 * 2**20 / 2e-3 / 1e12, 2)
    assert not any("GBps" in k or "copy" in k for k in e)


def test_speedups_name_their_base():
    entry = {k: {"ms": ms} for k, ms in (("fp32_mfma", 50.0), ("bf16x3", 25.0), ("bf16x3_k6", 20.0))}
    entry["gate_list_ms"] = 100.0
    bench.fused_speedups(entry)
    assert entry["bf16x3"] == {"ms": 25.0, "speedup_vs_gate_list": 4.0}
    entry["gate_by_gate_ms"] = 1000.0
    bench.fused_speedups(entry)
    assert entry["fp32_mfma"] == {"ms": 50.0, "speedup_vs_gate_list": 2.0, "speedup_vs_gate_by_gate": 20.0}
