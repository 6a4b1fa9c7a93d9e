"""The roofline block of the benchmark's line (no GPU needed): a rate over the HBM
peak is no bandwidth, so forms that take several steps per launch report none."""
import pytest

from test_bench_cpu import _bench_module


@pytest.mark.parametrize("name,streaming,bytes_per_step,steps,ms", [
    ("d2q9_shear2048_f32_fluid", "pull", 72 * 2048 ** 2, 500, 15.6),     # 135k MLUPS: 9.7 TB/s of the peak's 8
    ("d3q19_tgv256_f32_fluid", "push", 152 * 256 ** 3, 100, 29.8),
    ("d3q27_tgv192_f32_field", "pull", 228 * 192 ** 3, 100, 24.0)])
def test_several_steps_per_launch_have_no_bandwidth(name, streaming, bytes_per_step, steps, ms):
    r = _bench_module().roofline(name, streaming, "auto", bytes_per_step, steps, ms)
    assert all(r[k] is None for k in ("bound", "achieved", "frac", "traffic", "per_launch"))
    assert r["bytes_per_step_GB"] == round(bytes_per_step / 1e9, 4) and r["peak"] == 8000.0


@pytest.mark.parametrize("name,streaming,steps,launches", [
    ("d3q19_tgv256_f32dev_fluid", "aa", 100, 100), ("d3q19_tgv256_f32dev_fluid", "aa", 99, 100),
    ("d3q19_tgv256_f16dev_fluid", "pull", 100, None), ("d3q19_tgv256_f32_fluid_rawbasis", "pull", 100, None)])
def test_one_step_per_launch_reports_its_bandwidth(name, streaming, steps, launches):
    bench = _bench_module()
    r = bench.roofline(name, streaming, "auto", 2.55e9, steps, 41.3)
    assert r["bound"] == "hbm" and r["traffic"] == bench.TRAFFIC_GB[name, streaming]
    assert abs(r["achieved"] - 2.55 * steps / 41.3e-3) <= 0.05 and abs(r["frac"] - r["achieved"] / 8000.0) <= 1e-4
    assert (r["per_launch"] or {}).get("launches") == launches
