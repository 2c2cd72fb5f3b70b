"""Runtime code of the library on a host runtime (tests/host/hip_double.h), no
GPU: the built libigafd.so runs in a program that defines the HIP entry points
itself, so that waits, device allocations and launch limits can be looked at
and made to fail."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1602_01636_amd")


@pytest.fixture(scope="module")
def contexts(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(PKG, "libigafd.so")):
        pytest.skip("needs g++ and the built library")
    exe = str(tmp_path_factory.mktemp("host") / "contexts")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "host", "contexts.cpp"), "-o", exe, "-L" + PKG, "-ligafd",
           "-Wl,-rpath," + PKG, "-Wl,-rpath-link,/opt/rocm/lib", "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-3000:] + res.stderr[-3000:]
    return exe


def _check(exe, what):
    res = subprocess.run([exe, what], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.strip().endswith("OK"), (what, res.returncode, res.stdout[-2000:],
                                                                       res.stderr[-2000:])


@pytest.mark.parametrize("what", ["destroy_waits", "destroyed_stream"])
def test_memory_is_handed_on_after_its_stream(contexts, what):
    _check(contexts, what)


@pytest.mark.parametrize("what", ["cache_fit", "cache_holds_all", "cache_bound_and_age", "cache_failed_allocation", "cache_release"])
def test_block_cache(contexts, what):
    _check(contexts, what)


def test_release_is_bound():
    import paper_1602_01636_amd as api
    assert api.igafd_release_cached() >= 0
    assert api.igafd_release_cached() == 0


def test_decompositions_share_their_threads(contexts):
    _check(contexts, "eigen_budget")


def test_out_of_host_memory_is_a_status(contexts):
    _check(contexts, "host_memory")


def test_lds_limits_do_not_depend_on_the_problem(contexts):
    _check(contexts, "lds_limits")


def test_adi_lines_by_the_device(contexts):
    _check(contexts, "adi_lines")


def test_adi_setup_takes_two_allocations(contexts):
    _check(contexts, "adi_setup")


def test_tile_shape_without_room(contexts):
    _check(contexts, "tile_without_room")


def test_out_of_device_memory_is_a_status(contexts):
    _check(contexts, "device_memory")
