"""Host logic of the library that the real runtime cannot be made to exercise on demand -- its errors,
its capture state, sizes that no card holds -- on a stand-in runtime (fake_hip/), on the CPU.  Every
test runs in a process of its own: the stand-in has to be loaded in front of the real runtime."""

import os
import shutil
import subprocess
import sys

import pytest

from paper_2601_11590_amd import build

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "fake_hip")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no C++ compiler"
    subprocess.run([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", out], check=True)
    return out


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shim") / "libgemm_shim.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([shutil.which("g++") or "c++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    "-I" + build.CSRC, os.path.join(HERE, "gemm_shim.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("name", ["hash_plain", "pinned_memory_is_taken_at_create_and_the_bookkeeping_calls_nothing",
                                  "partial_hashes_lie_in_coherent_memory", "hash_with_an_uncollected_error",
                                  "hash_after_a_failed_launch", "hash_after_a_failed_wait", "hash_on_a_capturing_stream",
                                  "cached_hits_beside_an_uncollected_error", "launches_stay_within_the_thread_limit"])
def test_on_the_stand_in_runtime(fake, name):
    r = subprocess.run([sys.executable, os.path.join(HERE, "driver.py"), fake, build.library_path(), name],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "passed " + name in r.stdout, r.stdout[-3000:]


@pytest.mark.parametrize("name", ["gathered_gemm_reads_past_its_weights_only_where_allowed", "rotary_table_rule_counts_the_units_of_the_stream",
                                  "rows_behind_the_last_full_round"])
def test_gemm_launches_on_the_stand_in_runtime(fake, shim, name):
    r = subprocess.run([sys.executable, os.path.join(HERE, "driver.py"), fake, build.library_path(), name, shim],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "passed " + name in r.stdout, r.stdout[-3000:]
