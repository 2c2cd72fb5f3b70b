"""The thread team of the univariate eigensolver (host only, no GPU): bit for
bit the results of one thread, and free of data races under the thread
sanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1602_01636_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _run(tmp_path, flags, args, **kw):
    exe = str(tmp_path / "eigen_team")
    cmd = ["g++", "-std=c++17", *flags, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(ROOT, "tests", "host", "eigen_team.cpp"),
           os.path.join(CSRC, "setup1d.cpp"), "-o", exe, "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    res = subprocess.run([exe, *args], capture_output=True, text=True, timeout=600, **kw)
    if "unexpected memory mapping" in res.stderr:
        pytest.skip("the sanitizer's runtime does not start under this kernel's address layout")
    assert res.returncode == 0 and res.stdout.strip().endswith("OK"), res.stdout[-2000:] + res.stderr[-4000:]


def test_team_results_are_those_of_one_thread(tmp_path):
    _run(tmp_path, ["-O2"], [])


def test_team_under_the_thread_sanitizer(tmp_path):
    _run(tmp_path, ["-O2", "-g", "-fsanitize=thread"], ["600"],
         env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
