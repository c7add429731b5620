"""bench.py's figures of levels that run as one launch (no GPU): they count
what the factored products need, against the units that make them."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_levels_mod", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


STATS = dict(nodes=[0, 0, 50, 600, 500, 400, 300], iters_level=[0, 0, 100, 1000, 2000, 3000, 4000])
TIMING = dict(corr_ms=[0] * 7, select_ms=[0] * 7, level_ms=[0, 0, 0.01, 0.1, 0.3, 1.0, 3.0], steps=[0] * 7)


@pytest.mark.parametrize("prec", [0, 1])
def test_small_levels_count_their_own_products(bench, prec):
    """N = 16: 20 N^3 a node and 2 N^2 a step; N = 8: six products of 4 N^3 a
    step; both against the 16-bit matrix peak in either form.  N = 4 is the
    unfactored FP64 product."""
    r = bench.roofline(STATS, TIMING, prec, lambda n: f"k<{n}>", workload="none")
    lv = r["per_level"]
    for n, ops, ms in ((16, 20 * 16 ** 3 * 500 + 2 * 16 ** 2 * 2000, 0.3), (8, 6 * 4 * 8 ** 3 * 1000, 0.1)):
        assert lv[str(n)]["flops"] == ops and lv[str(n)]["peak"] == bench.PEAK_BF16_TFLOPS
        assert lv[str(n)]["frac"] == pytest.approx(ops / (ms * 1e-3) / 1e12 / bench.PEAK_BF16_TFLOPS, abs=1e-4)
    assert lv["4"]["peak"] == "fp64"
    assert lv["4"]["frac"] == pytest.approx(4 * 4 ** 4 * 100 / 0.01e-3 / 1e12 / bench.PEAK_FP64_TFLOPS, abs=1e-4)


def test_largest_level_figures_name_their_peak(bench):
    whole = bench.largest_level_figures(bench.roofline(STATS, TIMING, 0, lambda n: f"k<{n}>", workload="none"))
    assert set(whole) == {"level_tflops", "level_frac_16bit_peak"}
    step = dict(TIMING, corr_ms=[0, 0, 0, 0, 0, 0.5, 2.0], select_ms=[0, 0, 0, 0, 0, 0.4, 0.6], steps=[0] * 5 + [32, 32])
    r = bench.roofline(STATS, step, 0, lambda n: f"k<{n}>", workload="none")
    assert bench.largest_level_figures(r) == dict(corr_tflops=r["achieved"], corr_frac_fp32_peak=r["frac"])
    assert r["peak"] == bench.PEAK_FP32_TFLOPS
