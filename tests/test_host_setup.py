"""Set-up and first uses of a context without a GPU: api.cpp and eig1d.cpp are built with g++ (AddressSanitizer and
UndefinedBehaviorSanitizer) against stand-ins for the HIP runtime and the kernels' launch functions
(tests/host/setup_check.cpp), which keep an account of memory, filled arrays and queued work and can fail at any call."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_07711_amd", "csrc")
ROCM_INC = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INC), reason="g++ or the ROCm headers missing")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("setup") / "setup_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INC, "-I" + CSRC,
           os.path.join(ROOT, "tests", "host", "setup_check.cpp"), os.path.join(CSRC, "api.cpp"),
           os.path.join(CSRC, "eig1d.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300)

    def run(what):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=300, env=env)
        assert r.returncode == 0, (r.stdout[-3000:], r.stderr[-3000:])
        assert r.stdout.strip().endswith("ok") and not r.stderr
    return run


def test_setup_leaves_no_queued_work(program):
    program("waits")


def test_a_failed_call_leaves_nothing_half_made(program):
    program("faults")


def test_matrices_are_uploaded_once(program):
    program("uploads")


def test_a_small_context_is_small(program):
    program("memory")
