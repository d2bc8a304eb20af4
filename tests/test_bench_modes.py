"""Modes of the benchmark script that need no GPU to form their results."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_script", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_valu_mode_relates_the_rate_to_the_published_one():
    class Lib:
        @staticmethod
        def valu_rate(op):
            return 39.3e12 if op == "fma" else 9.825e12  # 78.6 TFLOP/s: every unit at 2.4 GHz

    r = _bench().mode_valu(Lib)
    assert abs(r["fma_over_published_78_6"] - 1.0) < 1e-12
    assert abs(r["transcendental_over_fma"]["rsq"] - 0.25) < 1e-12
