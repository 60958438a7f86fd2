"""The host half of packing a state on the CPU, against a stand-in for the
GPU runtime (tests/pack_runtime.cpp): which GPUs it may use for the
completed-parent lists, which clusters the row kernels take, and allocations
that fail.  The program defines the HIP calls that the library
makes, so the library under test is the built one."""

import os
import subprocess

import pytest

from paper_2605_07238_amd import build, fate

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("pack_runtime") / "pack_runtime")
    lib = os.path.abspath(fate.LIB_PATH)
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-g", "-std=c++17", "-I", build.INCLUDE,
                    "-I", build.CSRC, os.path.join(HERE, "pack_runtime.cpp"), "-x", "none", lib, "-o", out,
                    "-Wl,-rpath," + os.path.dirname(lib), "-Wl,--allow-shlib-undefined"], check=True)
    return out


def _run(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.returncode, r.stdout[-2000:], r.stderr[-2000:])


def test_lists_are_built_on_the_gpu_of_the_buffers_only(program):
    """The kernel runs where the DAGs, the buffer, the stream and the current
    device are one GPU; packing onto another GPU than the stream's, or from
    DAGs elsewhere, copies only.  The image is the host layout's either way."""
    _run(program, "devices")


def test_a_failed_allocation_reaches_the_caller(program):
    """Whichever allocation of a call fails, on whichever thread, the call ends
    with std::bad_alloc on the caller's thread or succeeds; never by aborting."""
    _run(program, "memory")


def test_clusters_that_the_row_kernels_take(program):
    """The row kernels' tables grow to just what fits the LDS, not past it."""
    _run(program, "shapes")
