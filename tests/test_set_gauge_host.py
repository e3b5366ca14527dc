"""Host test of wd_set_gauge's allocations (tests/set_gauge_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_set_gauge_allocations(tmp_path):
    exe = tmp_path / "set_gauge_check"
    # the launchers that these calls do not reach stay unresolved
    cmd = ["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
           "-Wno-unused-result", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1810_04201_amd", "csrc"),
           os.path.join(ROOT, "tests", "set_gauge_check.cpp"), "-o", str(exe),
           "-Wl,--unresolved-symbols=ignore-in-object-files"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = {k: v for k, v in os.environ.items() if not k.startswith("WD_")}
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120, env=env)
    assert out.returncode == 0 and out.stdout.strip().endswith("OK"), out.stdout + out.stderr
