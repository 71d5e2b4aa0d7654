"""Device memory as the library's host code handles it -- the tile workspace
made by a first product, and what is kept for later calls -- compiled with g++ against a HIP runtime that only
keeps count (tests/host/fake_hip.h); no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1902_01829_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")


def _program(tmp, name, sources):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp / name)
    subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-I" + HOST,
                    os.path.join(HOST, name + ".cpp"), *[os.path.join(CSRC, s) for s in sources], "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    return exe


def _check(exe, what, **env):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=60, env={**os.environ, **env})
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.fixture(scope="module")
def first_call(tmp_path_factory):
    return _program(tmp_path_factory.mktemp("host"), "matmat_first_call", ["h2_run.cpp"])


def test_first_fp64_columns_beside_another_streams_capture(first_call):
    _check(first_call, "beside_a_capture")


def test_fp64_columns_without_memory_for_tiles(first_call):
    _check(first_call, "no_memory")


def test_fp64_columns_take_the_memory_kept_for_later(first_call):
    _check(first_call, "memory_kept")


@pytest.fixture(scope="module")
def kept(tmp_path_factory):
    return _program(tmp_path_factory.mktemp("host"), "kept_memory", ["h2_api.cpp"])


def test_kept_memory_serves_its_own_size(kept):
    _check(kept, "sizes")


@pytest.mark.parametrize("what", ["bound", "given_back", "release", "short_memory"])
def test_memory_kept_for_later_calls(kept, what):
    """At most 1 GiB, of sizes that are asked for; all given back with the last
    handle, on request, and where the device is short of memory."""
    _check(kept, what)
