"""The field transfers' host side on the CPU (hostcopy_host.cpp: the library's
source file against a runtime that executes every call at once), in the
conditions that a GPU run does not bring about by itself."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("hostcopy") / "hostcopy_host")
    r = subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17",
                        os.path.join(HERE, "hostcopy_host.cpp"), "-o", out, "-lpthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


@pytest.mark.parametrize("case", ["launch_error", "no_memory", "forked_child", "short_lived",
                                  "large_first", "no_copy_engine"])
def test_host_transfers(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (case, r.returncode, r.stdout[-2000:], r.stderr[-2000:])
