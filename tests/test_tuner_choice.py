"""The autotuner's choice is not changed by one disturbed measurement (CPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_one_disturbance_does_not_change_the_choice(tmp_path):
    out = str(tmp_path / "fastest_host")
    r = subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(HERE, "fastest_host.cpp"), "-o",
                        out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
