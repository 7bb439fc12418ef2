"""The line that bench.py prints: short, with the keys its readers look for,
whatever the forms carry; and the compact schedule's byte counts, from which
its rates are made (CPU only)."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
            "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config")


def _line():
    big = {"workload": "w" * 200, "mlups": 12345.6, "kernels": {"pull": {"avg_ms": 0.1, "gbs": 1.0}},
           "autotune_ms": [0.1234] * 14, "mass_drift": [1e-16, -2e-16], "vs_fp32": {"u": 1e-3}}
    line = {k: "x" * 40 for k in CONTRACT}
    line.update(value=22338.1, vs_baseline=None, config={"workload": "w" * 90, "nodes": 1},
                roofline={"bound": "alu", "frac": 0.72, "hbm": {"frac": 0.49}, "kernel": "k" * 60},
                repeats={"mlups": [1.0] * 5, "median_mlups": 22300.1}, kernels=big["kernels"],
                cpu_baseline={"value": 4.26, "sample": "s" * 120, "threads1": {"value": 0.29}})
    forms = {f: dict(big) for f in bench.DEFAULT_FORMS.split(",")}
    for f in ("c3", "c5"):
        forms[f] = {"workload": "w" * 100, "fp32": dict(big), "fp16": dict(big), "bf16c": dict(big)}
    forms["table2"] = {"cases": [{"gamma": 1, "E_percent": 0.3}] * 8}
    forms["parity"] = {"c1": {"fp32_compact": {"e_rho": 1e-6, "status": "pass"}}}
    line["forms"] = forms
    line["parity_status"] = {"c1": {"fp32_compact": "pass"}, "c2": {"fp16": "fail"}}
    return line


def test_printed_line_is_short_and_complete():
    line = _line()
    text = json.dumps(bench.short_line(line))
    assert len(text) < 4000 and "\n" not in text, len(text)
    got = json.loads(text)
    for k in CONTRACT + ("roofline", "cpu_baseline"):
        assert got[k] == line[k], k
    assert got["repeats_median_mlups"] == 22300.1
    assert got["forms_mlups"]["fp16"] == 12345.6
    assert got["forms_mlups"]["c3"] == {"fp32": 12345.6, "fp16": 12345.6, "bf16c": 12345.6}
    assert "table2" not in got["forms_mlups"] and "parity" not in got["forms_mlups"]
    assert got["parity"] == {"runs": 2, "failed": ["c2/fp16"]}


def test_line_without_forms():
    line = _line()
    del line["forms"], line["parity_status"], line["cpu_baseline"]
    got = bench.short_line(line)
    assert all(got[k] == line[k] for k in CONTRACT) and "forms_mlups" not in got


@pytest.mark.parametrize("storage,pops,rho", [("fp32", 54 * 4, 0), ("fp32p", 54 * 4, 0),
                                              ("fp32x", 52 * 4 + 16, 16), ("fp16", 52 * 2 + 16, 16),
                                              ("bf16c", 52 * 2 + 16 + 2, 16)])
def test_byte_counts_of_the_compact_schedule(storage, pops, rho):
    """12 floats of the compact state and 11 moments, with the FP64 densities
    in both where the storage carries them."""
    step = 12 * 4 + 11 * 4 + 2 * rho
    want = {"pull": step, "fused": step, "pull_first": pops + 11 * 4 + rho,
            "emit": 12 * 4 + rho + pops}
    assert bench.compact_bytes(storage) == want
