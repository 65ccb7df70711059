"""The benchmark's printed line stays short enough to be kept whole by a
record of its last kilobytes, with the headline unabridged."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _kernel(bound):
    return {"bound": bound, "achieved": 5123.456789012345, "peak": 8000.0, "unit": "GB/s", "frac": 0.6404320986265431,
            "traffic": 1.951234567, "avg_launch_ms": 0.4712345678, "launches_per_step": 41.0}


def _record():
    config = {"workload": "uniform-1M-n64", "N": 1000000, "configurations": 1, "elements": "64^3", "L": 1.0,
              "screen": "one-element q=3", "mesh_order": 5, "near_block": "7^3", "outputs": "U, F", "precision": "fp64",
              "mg_rtol": 1e-7, "solver": "multigrid PCG", "boundary": "periodic", "near_pairs_per_step": 1308457448}
    kernels = {"near-screen field (FFTs + spectrum product)": _kernel("hbm"), "k_pair (near-pair sum)": _kernel("alu"),
               "k_apply p=5 (fine-level operator)": _kernel("hbm"),
               "transposed near field (FFTs + spectrum product)": _kernel("hbm")}
    stages = {f"a_stage_name_{k}": 12.345678901234567 for k in range(16)}
    variant = {"ms_per_step": 16.069263000000927, "value": 81426101993.59637, "stages_ms_per_step": stages,
               "kernel_fracs": dict.fromkeys(kernels, 0.1234), "accuracy_vs_fp64": {"Phi_rel_rms": 1.234567e-9}}
    return {"metric": "pair interactions/s + N=1M energy+force time at 1e-6 rel. RMS err vs Ewald",
            "value": 40612345678.123456, "unit": "pair interactions/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 32.21987654321, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
            "data": "synthetic", "config": config, "roofline": dict(_kernel("hbm"), kernel="k_apply p=5 (fine-level operator)"),
            "kernels": kernels, "stages_ms_per_step": stages, "mg_iterations": 5, "adj_mg_iterations": 5,
            "mg_rel_residual": 3.7503741051149e-08, "create_seconds": 0.172110982, "practical_hbm_gbs": 5031.234567,
            "pair_variant": {}, "U": [1.0], "hbm_stages": {"kernels": kernels},
            "variants": {f"mixed a-workload-of-1M-n64 with options {k:02d}": variant for k in range(22)},
            "screen_sweep": {"rows": [{"screen": "27-element q=3", "near_block": f"{k}^3", "ms_per_step": 129.123456789,
                                       "ewald": {"Phi_rel_rms": 3.791234e-05}} for k in range(8)]},
            "method_error_vs_ewald": {"reference": "Ewald (oracle)", "Phi_rel_rms": 1.2e-6, "F_rel_rms": 2.3e-6},
            "method_error_vs_ewald_full_size": {"reference": "r" * 400, "Phi_rel_rms": 1.2e-6, "F_rel_rms": 2.3e-6},
            "cpu_baseline": dict({f"a_measured_number_{k}": 2446.466485997002 for k in range(10)}, note="n" * 600)}


def test_printed_line_is_short_and_keeps_the_headline():
    import bench

    rec = _record()
    assert len(json.dumps(rec)) > 16000       # what a run measures
    text = json.dumps(bench.headline(rec))
    assert len(text) < 4000 and "\n" not in text
    line = json.loads(text)
    for k in bench.HEADLINE:
        assert line[k] == rec[k], k
    assert line["roofline"]["kernel"] == rec["roofline"]["kernel"] and len(line["variants_ms"]) == 22
    assert len(line["screens_ms_err"]) == 8


def test_printed_line_of_a_plain_run():
    import bench

    rec = _record()
    for k in ("variants", "screen_sweep", "cpu_baseline", "method_error_vs_ewald", "method_error_vs_ewald_full_size",
              "hbm_stages"):
        del rec[k]
    line = bench.headline(rec)
    assert set(bench.HEADLINE) <= set(line) and "variants_ms" not in line
