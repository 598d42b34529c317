"""The benchmark's JSON line stays short enough to be read whole from the end of
an output."""
import importlib.util
import json
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_line_is_short():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    roof = {"bound": "alu", "achieved": 23.489937358086255, "peak": 78.6, "unit": "TFLOP/s", "frac": 0.2988541648611483,
            "traffic": 1.23456789e9, "traffic_source": "x" * 80, "kernel": "jk_k1_row<1, 0, 0, 0, double, 256>"}
    build = {f"figure_{k}": 1234.56789012345 / (k + 1) for k in range(18)}
    build |= {"roofline": roof, "vs_oracle": {f"max_{k}": 3.4611202792689255e-13 for k in range(6)},
              "top_kernels": [{"kernel": "k" * 40, "ms_per_build": 12.309320397675037, "tflops": 23.48} for _ in range(12)]}
    configs = {c: {"workload": "w" * 100, "fp64": build, "mixed": build} for c in ("c1", "c2", "c4", "qz8")}
    assert len(json.dumps(configs)) > 14000
    short = bench.compact(configs)
    assert len(json.dumps(short)) < 8000
    assert short["c1"]["fp64"]["figure_1"] == 617.28 and "top_kernels" not in short["c2"]["mixed"]
    assert short["qz8"]["fp64"]["roofline"] == {"kernel": roof["kernel"], "achieved": 23.49, "frac": 0.29885}
