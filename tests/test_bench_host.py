"""bench.py's command-line contract on the host (no GPU needed)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    """--gpus above 1 exits with status 2 and says why, before touching a GPU."""
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 2
    assert "one GPU only" in r.stderr
    assert r.stdout.strip() == ""


def test_alu_peak_by_precision():
    """256 CUs x 4 SIMDs x 64 lanes x 2 operations x 2.4 GHz, over two cycles an
    instruction in FP32 and four in FP64."""
    sys.path.insert(0, ROOT)
    import bench
    for precision, cycles in (("fp32", 2), ("fp64", 4)):
        peak = 256 * 4 * 64 * 2 * 2.4e9 / cycles * 1e-12
        assert abs(bench.ALU_PEAK_TFLOPS[precision] / peak - 1) < 1e-3
