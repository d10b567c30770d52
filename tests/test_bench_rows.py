"""What bench.py's rows say: a rate at which single steps would move memory is not called memory
bandwidth, and the adjoint's forward reference is one step per launch, as an adjoint step is."""
import importlib.util
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_rows", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    sys.modules["bench_rows"] = m
    spec.loader.exec_module(m)
    return m


def _times(source, name):
    body = source[source.index(f"def {name}("):]
    return body[:body.index("\ndef ")]


@pytest.mark.parametrize("name", ["measure_adjoint", "measure_adjoint_large"])
def test_forward_reference_is_single_steps(bench, name):
    body = _times(open(bench.__file__).read(), name)
    assert "fwd_ms = time_single_steps(" in body
    assert "graph" not in body


def test_line_is_short(bench):
    """A default run has 52 variants, whose rows in full made a line of 21 KB; of a program's
    output, its log included, 13 KB are commonly kept."""
    rows = [{"workload": f"reduced precision: porous discs 4096^2 phi=0.5, {k} steps", "dtype": dt,
             "layout": "dense_ab", "glups": 123.456789 + k, "ms_per_step": 0.1234567,
             "mass_drift": -1.23456789e-13, "l2_err_vs_fp64": 0.00123456789,
             "l2_err_reference": "FP64 HIP path, same layout and step count", "steps": 5000}
            for k in range(13) for dt in ("f64", "f32", "f16s", "bf16s")]
    short = bench.short_variants(rows)
    assert sum(len(v) for v in short.values()) == len(rows)
    assert short[rows[5]["workload"]]["f32 dense_ab"]["glups"] == 124.5
    assert len(json.dumps(short)) < 6000
    # rows without a rate of their own keep their time
    assert bench.short_variants([{"workload": "w", "ms_per_step": 2.0}]) == {
        "w": {"": {"ms_per_step": 2.0}}}


@pytest.mark.gpu
def test_rows(bench):
    import paper_2108_13241_amd as lbm
    import synthetic
    row = bench.measure_dense(lbm, 512, "f32", "dense_ab", 20, 4, synthetic.taylor_green(512, 0.01))
    assert "hbm_gbps" not in row
    assert row["single_step_gbps"] == pytest.approx(row["glups"] * row["bytes_per_node"])

    class Lattice:
        calls = []

        def step(self, n):
            self.calls.append(n)

    bench.time_single_steps(Lattice(), 5, 3)
    assert Lattice.calls == [1] * 8
