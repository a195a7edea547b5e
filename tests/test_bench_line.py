"""The benchmark's printed line keeps the headline's keys and every workload's times, shapes
and errors, and stays short enough for a reader that keeps the end of the output."""
import json

import bench


def _form(x):
    return {"ms_per_step": x, "kernel_ms_mean": x, "kernel_ms_min": x, "tile": "0x8fo2", "tune_ms": x, "elements_per_s": 1e9 / x,
            "alg_flops_per_element": 1e6, "fdom_equiv_gflops": 1e5 / x, "gflops_alg": 1e5 / x, "tflops_frac_of_peak": x / 7,
            "hbm_gbs_algorithmic": 1e3 / x, "rel_err_A": x * 1e-7, "rel_err_A_max_elem": x * 1e-6, "rel_err_b": x * 1e-7,
            "rel_err_b_max_elem": x * 1e-6, "err_sample": "64 elements (every 256th)",
            "roofline": {"bound": "mfma", "peak": 78.6, "unit": "TFLOP/s", "achieved": x, "frac": x / 78.6, "traffic": None}}


def _line(forms):
    return {"metric": "m" * 100, "value": 1.234567890123e8, "unit": "elements/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 1.234567890123, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "d" * 60,
            "data": "synthetic (seeded perturbed prism mesh and coefficients)", "config": {"workload": "w", "p": 4, "note": "n" * 250},
            "fdom_equiv_gflops": 1.23456789e5, "roofline": {"bound": "mfma", "achieved": 1 / 3, "peak": 2500.0, "unit": "TFLOP/s",
                                                            "frac": 1 / 3, "traffic": None, "note": "n" * 150},
            "cpu_baseline": {"value": 1 / 7, "unit": "elements/s", "cores": 16, "kind": "oracle", "sample": "s" * 80},
            "forms": {f: _form(i + 1 / 3) for i, f in enumerate(forms)}, "device": "AMD Instinct MI355X"}


def test_brief():
    four = ["bf16x3", "fp16x3", "fp32", "fp64"]
    line = _line(four)
    line["configs"] = {n: bench.summarise(_line(four[2:])) for n in
                       ("p1_4096", "p1_524288", "adj_p3_131072", "adj_p7_16384", "tet_p4_393216")}
    line["configs"]["p7_16384"] = bench.summarise(_line(four))
    degrees = {f"p{p}": {f: {"sumfact": _form(p / 3), "xi3": _form(p / 7), "speedup_vs_xi3": 6.123} for f in four[2:]} for p in range(4, 8)}
    line["configs"]["hex_p4_p7"] = bench.summarise({**_line([]), "degrees": degrees})
    line["configs"]["laplace_paper_sweep"] = bench.summarise(
        {**_line([]), "degrees": {f"p{p}": {**_form(p / 3), "paper_convention_gflops": 1e6 / p} for p in range(1, 8)}})
    line["configs"]["mixed_262144"] = bench.summarise(
        {**_line([]), "graph_ms": 1 / 3, "persistent_ms": 1 / 3, "tile_sets_ms": {"v" * 26 + str(i): 1 / 3 for i in range(9)},
         "errors_vs_oracle": {f"p{p}": {"rel_err_A": p / 3e7, "rel_err_b": p / 3e7, "elements": 1024} for p in range(1, 7)}})
    out = bench.brief(line)
    text = json.dumps(out)
    assert len(text) < 7000 and json.loads(text) == out
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert out[k] == line[k]
    assert out["forms"]["fp64"] == [3.333, "0x8fo2", 3.333e-07, 3.333e-07] and set(out["configs"]) == set(line["configs"])
    for name, c in line["configs"].items():
        assert out["configs"][name]["value"] == float(f"{c['value']:.4g}") and "frac" in out["configs"][name]
    assert out["configs"]["hex_p4_p7"]["degrees"]["p7"]["fp32"]["sumfact"][0] == 2.333
    assert out["configs"]["mixed_262144"]["rel_err_A"][5] == 2e-7
