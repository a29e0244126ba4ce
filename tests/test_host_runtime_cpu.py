"""Host runtime (argument checks, workspaces, launch sequences, error returns) on a HIP runtime
of host memory: tests/cpp/host_check.cpp, under AddressSanitizer, one check per test."""
import os
import subprocess

import pytest

from tests.conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2406_06488_amd", "csrc")


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_check")
    cmd = ["/opt/rocm/bin/hipcc", "--offload-host-only", "-O1", "-g", "-std=c++17", "-Xarch_host",
           "-fsanitize=address", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "cpp", "host_check.cpp"), os.path.join(CSRC, "runtime.cpp"),
           os.path.join(CSRC, "baselines.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("build failed:\n" + r.stderr[-4000:])
    return exe


@pytest.mark.parametrize("check", ["failed_calls_wait", "failed_calls_free",
                                   "fork_of_two_devices", "staging_of_two_devices",
                                   "graphs_of_two_devices", "timing_of_two_devices",
                                   "plan_buffers"])
def test_host_runtime(host_check, check):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    out = subprocess.run([host_check, check], capture_output=True, text=True, env=env, timeout=120)
    assert out.returncode == 0, out.stdout[-4000:] + out.stderr[-4000:]
    assert out.stdout.strip() == "ok"
