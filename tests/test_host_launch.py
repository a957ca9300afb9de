"""CPU: what the library's host code asks of the kernels and the HIP runtime.  The
real jx_abi.cpp and jx_server.cpp run over stand-ins for both
(tests/sanitize/fake_hip.h), under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil

import pytest

from tests.test_host_sanitize import CSRC, ROOT, _build_and_run

ARGS = ["-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
        "-I/opt/rocm/include", os.path.join(CSRC, "jx_host.cpp"), os.path.join(CSRC, "jx_layout.cpp")]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_launch_mappings(tmp_path):
    out = _build_and_run(tmp_path, "g++", ARGS + [os.path.join(ROOT, "tests", "sanitize", "launch_checks.cpp")],
                         "launch_checks")
    assert "launch checks: 0 failures" in out


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_serving_loop(tmp_path):
    out = _build_and_run(tmp_path, "g++", ARGS + [os.path.join(ROOT, "tests", "sanitize", "server_checks.cpp")],
                         "server_checks")
    assert "server checks: 0 failures" in out
