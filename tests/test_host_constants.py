"""Constants of the kernels that others rely on: the sources do not compile when
one is changed without the other (no GPU; the device pass of hipcc checks the
syntax of a changed copy)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1602_01636_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")

pytestmark = pytest.mark.skipif(HIPCC is None, reason="needs hipcc")


def _compiles(tmp_path, source, old=None, new=None):
    text = open(os.path.join(CSRC, source)).read()
    if old:
        assert text.count(old) == 1, old
        text = text.replace(old, new)
    copy = tmp_path / source
    copy.write_text(text)
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-fsyntax-only",
                          "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), str(copy)],
                         capture_output=True, text=True, timeout=300)
    return res.returncode == 0, res.stderr


@pytest.mark.parametrize("source, old, new", [
    # copies of columns left of an edge tile land in the padding of the LDS rows
    ("gemm.hip", "constexpr int kPad = 16;", "constexpr int kPad = 4;"),
    ("gemm.hip", "constexpr int kGap = 16;", "constexpr int kGap = 2;"),
    # a training block adds the gradient images of its two waves
    ("mlp.hip", "return train ? 2 : kBlock / 64;", "return train ? 4 : kBlock / 64;"),
    # arguments of the element kernels' many small launches
    ("assembly.hip", "  const double* der[3];\n  int n[3];", "  const double* der[3];\n  const int* at[3];\n  int n[3];"),
])
def test_dependent_constants(tmp_path, source, old, new):
    ok, err = _compiles(tmp_path, source)
    assert ok, err[-2000:]
    ok, err = _compiles(tmp_path, source, old, new)
    assert not ok and "static assertion failed" in err, err[-2000:]
