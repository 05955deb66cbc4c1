"""The surrogate's reduction scratch holds what its kernels write, for every
shape pf_fno_create accepts (host arithmetic only)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_partial_sums_fit_their_scratch(tmp_path):
    exe = str(tmp_path / "fno_sizes_check")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-o", exe,
                        os.path.join(ROOT, "tests", "native", "fno_sizes_check.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.split() == ["ok", str(32 * 32 * 16 * 8 * 8)]
