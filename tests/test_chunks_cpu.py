"""The cuts of concatenated vectors into workgroups, on the host (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_chunks(tmp_path):
    exe = str(tmp_path / "chunks_check")
    r = subprocess.run(["hipcc", "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host", "chunks_check.cpp"),
                        os.path.join(ROOT, "paper_2107_09006_amd", "csrc", "k_krylov.hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr + r.stdout
    assert r.stdout.splitlines()[-1] == "OK"
