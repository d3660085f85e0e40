"""The rule that splits a prepared call's keys over the waves of 64-row units
(CPU only): ``keys_split`` in ``csrc/sol_internal.h``, compiled by the host
compiler.  One round of the 256 CUs always splits, a second one only over a long
walk: every key of a dense call or of a block-sparse one with prefix rows, longer
still where every query block walks a list; never a third."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_35110_amd", "csrc")

SRC = r'''
#include "sol_internal.h"
extern "C" int split(long long units, int n_keys, int all_listed) { return sol::keys_split(units, n_keys, all_listed); }
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the HIP headers not available")
    d = tmp_path_factory.mktemp("rule")
    src, so = str(d / "rule.cpp"), str(d / "librule.so")
    open(src, "w").write(SRC)
    res = subprocess.run([gxx, "-std=c++17", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__",
                          "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC, src, "-o", so],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    lib = ctypes.CDLL(so)
    lib.split.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    return lib


@pytest.mark.parametrize("units,n_keys,every_key,listed", [
    (1, 1, 1, 1), (256, 1, 1, 1), (256, 1 << 23, 1, 1),
    (257, 1791, 0, 0), (257, 1792, 1, 0), (512, 1792, 1, 0),
    (512, 4096, 1, 0), (512, 12287, 1, 0), (257, 12288, 1, 1), (512, 12288, 1, 1), (512, 1 << 23, 1, 1),
    (513, 1792, 0, 0), (513, 1 << 23, 0, 0), (1 << 40, 1 << 23, 0, 0)])
def test_rule(lib, units, n_keys, every_key, listed):
    assert lib.split(units, n_keys, 0) == every_key
    assert lib.split(units, n_keys, 1) == listed
