"""The lengths of a run's launches, unit-tested on the CPU with g++."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_take_the_time_meant_for_them(tmp_path):
    exe = tmp_path / "test_launch_length"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "cpp", "test_launch_length.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
