"""The benchmark's figures for the projection and for the rotation come from launches that do that work alone."""
import bench

WORK = {"qkv_flops": 2e11, "rerope_bytes": 1e8, "rerope_bytes_all": 1.2e8, "moved_bytes": 2e8, "moved_bytes_all": 2.4e8}


def _kern(**ms):
    return {k: {"launches_per_step": 1.0, "avg_ms": v, "ms_per_step": v} for k, v in ms.items()}


def test_one_launch_for_both():
    r = bench.projection_and_rotation_rates(_kern(qkv=0.25, attention=1.0), WORK, {"qkv": 2e-4, "rerope": 5e-5})
    assert abs(r["qkv_tflops"] - 1000.0) < 1e-9                       # 2e11 / 0.2 ms, not / 0.25 ms
    assert abs(r["rerope_gbs_algorithmic"] - 2400.0) < 1e-9 and abs(r["rerope_plus_vcopy_gbs_moved"] - 4800.0) < 1e-9
    assert abs(r["rerope_frac_of_hbm_peak"] - 0.3) < 1e-12
    both = r["qkv_with_rotation"]
    assert abs(both["tflops"] - 800.0) < 1e-9 and abs(both["gbs_moved"] - 800.0) < 1e-9 and both["ms"] == 0.25


def test_a_launch_each():
    r = bench.projection_and_rotation_rates(_kern(qkv=0.2, rerope=0.04), WORK, None)
    assert abs(r["qkv_tflops"] - 1000.0) < 1e-9 and abs(r["rerope_gbs_algorithmic"] - 2500.0) < 1e-9
    assert abs(r["rerope_plus_vcopy_gbs_moved"] - 5000.0) < 1e-9 and "qkv_with_rotation" not in r


def test_no_rotation_of_its_own():
    """Host pools are rotated by the stream-in kernel, which is timed as the rotation's class; r = 100 % rotates nothing."""
    r = bench.projection_and_rotation_rates(_kern(qkv=0.2), WORK, None)
    assert set(r) == {"qkv_tflops"} and abs(r["qkv_tflops"] - 1000.0) < 1e-9
    assert bench.projection_and_rotation_rates({}, WORK, None) == {}
