"""CPU: the library's host code on a stand-in for the HIP runtime (tests/native/hip_stub).

The stand-in executes no kernels; it keeps the order of the work on the streams, checks that every use and free
of device memory is ordered behind the work of other streams on it, and records the quadratures launched.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1609_08146_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")


@pytest.fixture(scope="session")
def host_checks(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "host_checks")
    src = [os.path.join(CSRC, f) for f in ("sc_api.cpp", "sc_serve.cpp", "sc_gauss_host.cpp")]
    src += [os.path.join(NATIVE, "hip_stub", "stub.cpp"), os.path.join(NATIVE, "host_checks.cpp")]
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(NATIVE, "hip_stub"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, *src, "-lquadmath", "-o", out], check=True)
    return out


@pytest.mark.parametrize("name", ["idle_blocks", "block_sizes", "block_turnover", "no_waits", "chunks", "batch_cap",
                                  "tuner", "other_device"])
def test_host_code(host_checks, name, tmp_path):
    r = subprocess.run([host_checks, name], capture_output=True, text=True, timeout=300, cwd=tmp_path)
    assert r.returncode == 0, r.stdout + r.stderr
