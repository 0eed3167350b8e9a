"""bench.py command line: the parts that need no GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    """Every box has one GPU and the build has no collectives: --gpus N with N > 1 exits with a message, no JSON line."""
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=300)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr + r.stdout
    assert "{" not in r.stdout


def _bench():
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    return bench


def test_the_convolution_rate_counts_packing_and_reduction():
    names = ["nsk_conv2d_pack_filters", "nsk_conv2d_fwd_stats", "nsk_bn_relu_add_fwd_mask", "nsk_conv2d_wgrad_partial", "nsk_conv2d_dgrad_packed", "nsk_conv2d_wgrad_reduce"]
    costs = [("p", 0.0, 0.0), ("f", 3e9, 1e6), ("b", 0.0, 1e6), ("w", 3e9, 1e6), ("d", 3e9, 1e6), ("r", 0.0, 0.0)]
    flops, ms = _bench().conv_totals(names, costs, [1.0, 2.0, 4.0, 8.0, 16.0, 32.0])
    assert flops == 9e9 and ms == 59.0


def test_the_roofline_names_the_unit_and_what_is_left_out():
    bench = _bench()
    conv = ("conv2d_fwd/dgrad", 9.664e9, 67.3e6, 0.075)
    large = bench.roofline("f32", *conv, {"nsk_conv2d_fwd_stats", "nsk_conv2d_dgrad"})
    assert large["bound"] == "mfma" and abs(large["peak"] - 2516.6 / 6) < 1e-9 and "not_in_launch" not in large
    assert abs(large["frac_of_f32_unit"] - 9.664e9 / 75e-6 / 157.3e12) < 1e-9
    small = bench.roofline("f32", "conv2d_fwd/dgrad", 3e7, 1e6, 0.01, {"nsk_conv2d_fwd"})
    assert small["peak"] == 157.3 and "frac_of_f32_unit" not in small
    split = bench.roofline("bf16", "conv2d_wgrad", 1e11, 1e6, 0.1, {"nsk_conv2d_wgrad_partial"})
    assert split["not_in_launch"] == ["addition of the partial sums (nsk_conv2d_wgrad_reduce)"]
    assert bench.roofline("f32", "bn_relu_add_fwd", 0.0, 1e8, 0.02, {"nsk_bn_relu_add_fwd_mask"})["bound"] == "hbm"
