"""The cache of device blocks on a stubbed allocator (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_device_blocks(tmp_path):
    exe = str(tmp_path / "blocks_check")
    r = subprocess.run(["hipcc", "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host", "blocks_check.cpp"),
                        os.path.join(ROOT, "paper_2107_09006_amd", "csrc", "blocks.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr + r.stdout
    assert r.stdout.splitlines()[-1] == "OK"
