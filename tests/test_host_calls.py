"""The library's host sources compiled with a plain C++ compiler against a
runtime that only counts (tests/host): bookkeeping that a device would hide or
that must not go wrong on one.  Host-only: no device is touched."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def _run(name, tmp_path, *args):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / name)
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2208_10859_amd/csrc", f"-I{HOST}",
                    os.path.join(HOST, name + ".cpp"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
    return r.stdout


def test_encoder_call_waits_for_its_kernels_also_after_an_error(tmp_path):
    """The encoder's kernels write the caller's planes and a workspace that
    outlives the call: no call may return while one of them runs."""
    _run("encode_calls", tmp_path)


@pytest.mark.parametrize("n", ["2", "4", "7"])
def test_encoder_calls_of_several_threads_run_side_by_side(tmp_path, n):
    """Threads with streams of their own on one context: no call waits for
    another, none shares a workspace or an overflow flag, and what the context
    keeps is bounded."""
    _run("encode_calls", tmp_path, n)


def test_tiles_of_mixed_levels_are_dealt_over_the_ranges_of_the_xcds(tmp_path):
    """Every launch size, with one to 32 work units per tile."""
    _run("deal_items", tmp_path)


def test_storage_order_by_counting_equals_the_sorted_one(tmp_path):
    """Every tile edge and level count, and the table of a frame's planes."""
    _run("storage_order", tmp_path)


def test_calls_take_the_strips_that_suit_their_number_of_tiles(tmp_path):
    """GOPs of 41 to 48 tiles and sets whose last round of 32-row strips is more
    than two thirds full run in those, other YUV420 calls in the 16-row ones; a
    chosen variant holds for every call."""
    _run("call_variant", tmp_path)
