"""The decode's host-side shape decisions (csrc/decode_plan.h), built with g++: every pair of
record sizes up to 128 bytes has a plan that fits the matrix-core kernel, at every number of query
heads per KV head."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "libplan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2608_14191_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "decode_plan_harness.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.plan_misfits.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.plan_of.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64] * 2 + [ctypes.c_int, ctypes.c_void_p]
    return lib


@pytest.mark.parametrize("G", range(1, 17))
def test_every_pair_of_records_has_a_plan(lib, G):
    for kv_rows in (1, 8, 64, 320):
        for cap in (64, 1024, 32768, 1 << 20):
            for append in (0, 1):
                assert lib.plan_misfits(G, kv_rows, cap, append) == 0, (kv_rows, cap, append)


@pytest.mark.parametrize("rk,rv,G,append,nt,hg,ntile,fused", [
    (44, 44, 4, 1, 1, 1, 8, 1), (44, 44, 8, 1, 2, 1, 8, 1), (44, 44, 9, 1, 2, 2, 8, 0),
    (96, 96, 8, 1, 2, 1, 4, 1), (100, 96, 5, 1, 1, 2, 4, 0), (128, 128, 4, 1, 1, 1, 4, 1),
    # values much wider than the keys: four heads per workgroup, or 512 tokens
    (64, 96, 7, 1, 1, 2, 4, 0), (64, 96, 4, 1, 1, 1, 4, 1), (36, 96, 16, 0, 1, 4, 4, 0),
    (24, 64, 12, 0, 2, 2, 4, 0), (32, 64, 12, 0, 2, 2, 8, 0)])
def test_chosen_plans(lib, rk, rv, G, append, nt, hg, ntile, fused):
    f = ctypes.c_int()
    p = lib.plan_of(rk, rv, G, 64, 32768, append, ctypes.byref(f))
    assert (p & 255, p >> 8 & 255, p >> 16 & 255, f.value) == (nt, hg, ntile, fused)
