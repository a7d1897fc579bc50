"""bench.py contract checks that need no GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode != 0
    assert "one GPU" in res.stderr
    assert res.stdout.strip() == ""


def test_help_lists_the_contract_flags():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--help"], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0
    for flag in ("--gpus", "--steps", "--warmup", "--workload"):
        assert flag in res.stdout


def test_named_backward_kernels_follow_the_library_rules():
    # the same points of the rules as the host test of the library pins (one pass or two, order of the passes)
    import bench
    name = bench._backward_kernels
    assert name([256] * 85, 1, 128) == "bwd_prepare_kernel + attn_bwd_both_kernel"
    assert name([256] * 86, 1, 128) == name([256], 1, 64) == name([96], 1, 128) == "attn_bwd_fused_kernel"
    assert name([128], 128, 128).endswith("attn_bwd_both_kernel") and name([128], 129, 128) == "attn_bwd_fused_kernel"
    assert "bwd_short_delta_kernel" in name([300, 20], 4, 128) and "both" in name([1024], 32, 128)
    assert name([56320], 32, 128) == "attn_bwd_dq2_kernel + attn_bwd_dkdv_kernel"
    assert name([1000, 1], 2, 64) == "bwd_prepare_kernel + bwd_short_delta_kernel + attn_bwd_dkdv_kernel + attn_bwd_dq_kernel"
    assert [bench._temporal_backward_kernels(t)[:6] for t in (16, 17, 128, 129)] == ["tattn_", "tattnB", "tattnB", "tattnL"]
