"""The decode's host-side shape decisions (csrc/decode_plan.h), built with g++: every pair of
record sizes up to 128 bytes has a plan that fits the matrix-core kernel, at every number of query
heads per KV head."""
import ctypes
import heapq
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


def _deal(lib, nch, rps, chunks):
    arr = (ctypes.c_int * len(nch))(*nch)
    grid, runs = ctypes.c_int64(), ctypes.c_int()
    lib.runs_of.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
                            ctypes.c_void_p, ctypes.c_void_p]
    q = lib.runs_of(arr, len(nch), rps, chunks, ctypes.byref(grid), ctypes.byref(runs))
    return q, grid.value, runs.value


def _rounds(lib, nch, rps, q, grid, runs):
    """The time of the dealt runs in chunk times: every XCD's 32 compute units take its workgroups
    in order, a run costs its chunks and one more."""
    length = []
    for c in nch:
        n = -(-c // q)
        length += ([q] * (n - 1) + [c - (n - 1) * q]) * rps   # (order within a sequence: any)
    units = [[0.0] * 32 for _ in range(8)]
    for heap in units:
        heapq.heapify(heap)
    for block in range(grid):
        r = lib.block_run(block, runs)
        if r >= 0:
            heap = units[block % 8]
            heapq.heapreplace(heap, heap[0] + length[r] + 1)
    return max(max(h) for h in units)


LENGTHS = {"even": lambda i, b, n: n, "third": lambda i, b, n: max(1, n - i * 2 * n // (3 * b)),
           "random": lambda i, b, n: 1 + (7919 * i + 13 * n) % n, "one": lambda i, b, n: n if i == 0 else 1,
           "two": lambda i, b, n: n if i % 2 else max(1, n // 2)}


@pytest.mark.parametrize("rps", [4, 8, 16])
@pytest.mark.parametrize("kind", list(LENGTHS))
def test_runs_of_a_ragged_batch(lib, kind, rps):
    for b in list(range(2, 20)) + [24, 31, 32, 33, 40, 48, 65, 70, 130]:
        for n in (1, 2, 3, 5, 8, 16, 33, 64, 128):
            nch = [LENGTHS[kind](i, b, n) for i in range(b)]
            rows, chunks = b * rps, 2 * n                # (capacity above the longest)
            if rows * chunks <= 256:
                continue                                 # (dealt evenly)
            q, grid, runs = _deal(lib, nch, rps, chunks)
            count = rps * sum(-(-c // q) for c in nch)
            assert grid % 8 == 0 and rows <= grid <= max(256, rows + 512) and runs == count <= grid
            blocks = [lib.block_run(i, runs) for i in range(grid)]
            assert sorted(x for x in blocks if x >= 0) == list(range(runs))
            share = [sum(x >= 0 for x in blocks[x8::8]) for x8 in range(8)]
            assert max(share) <= -(-runs // 8)
            # no worse than a workgroup for every chunk, which repeats the planes and the merge
            # (two chunk times each); one long sequence among one-chunk ones fills one XCD first
            rounds = -(-rps * sum(nch) // 256)
            slack = 1.8 if kind == "one" else 1.1
            assert _rounds(lib, nch, rps, q, grid, runs) <= slack * 2 * rounds + 1, (b, n, q, grid, runs)


@pytest.mark.parametrize("batch,rows,chunks,even", [
    (1, 8, 4096, 1), (4, 32, 8, 1), (4, 32, 9, 0), (64, 512, 1, 1), (64, 512, 2, 0), (40, 320, 1, 1),
    (128, 1024, 4, 1), (128, 1024, 5, 0), (1000, 1000, 2, 0), (2048, 16384, 64, 1)])
def test_rows_that_wait_for_no_length(lib, batch, rows, chunks, even):
    """Rows of one chunk, however many, and many rows of few chunks are dealt without the lengths."""
    lib.dealt_evenly.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    assert lib.dealt_evenly(batch, rows, chunks) == even


def test_quotients_of_runs(lib):
    """The run count of a row without an integer division, over all its range."""
    lib.wrong_quotients.restype = ctypes.c_int64
    for n_max, q_max, step_n, step_q in ((4096, 4096, 1, 1), (1 << 20, 1 << 20, 9973, 8191)):
        assert lib.wrong_quotients(n_max, q_max, step_n, step_q, 2) == 0
