"""The benchmark's line stays short enough to be read from the end of its output, whatever the legs report."""

import json

import bench

HEAD = {"metric": "m", "value": 472764.33687071, "unit": "gate updates/s", "n_gpus": 1, "steps": 20, "warmup": 5,
        "ms_per_step": 6.091830062866211, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "c64+f64",
        "data": "synthetic", "config": {"workload": "eagle127_d16", "instances": 1}}


def _leg():
    return {"workload": "w", "value": 1000566.7737921913, "ms_per_evolution": 92.10779571533203, "max_abs_err_vs_oracle": 3.8120454e-05,
            "all_within_max_1e-5_8S": True, "kernels": {f"k{i}": {"avg_ms": 0.1 + i} for i in range(9)},
            "roofline": {"frac": 0.0189329414, "unit": "TFLOP/s"}, "sample": "x" * 200,
            "max_abs_err_vs_oracle_per_instance": [1.234e-07 * i for i in range(256)]}


def test_figures_are_kept_and_lists_are_not():
    out = dict(HEAD, d32_sweep=_leg(), infinite_lattice=_leg())
    text = bench.result_line(out)
    got = json.loads(text)
    assert "\n" not in text and len(text) <= bench.LINE_LIMIT
    assert {k: got[k] for k in HEAD} == HEAD
    for leg in ("d32_sweep", "infinite_lattice"):
        assert got[leg] == {"workload": "w", "value": 1000570.0, "ms_per_evolution": 92.1078, "max_abs_err_vs_oracle": 3.81205e-05,
                            "all_within_max_1e-5_8S": True, "roofline_frac": 0.01893}


def test_any_number_of_legs_fits():
    text = bench.result_line(dict(HEAD, **{f"leg{i}": _leg() for i in range(100)}))
    got = json.loads(text)
    assert len(text) <= bench.LINE_LIMIT and {k: got[k] for k in HEAD} == HEAD and "leg0" in got
