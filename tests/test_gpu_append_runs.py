"""The fused append at every number of runs per row where its coefficients are shared out
differently (one run, two or three, up to 31, 32 and more), and short contexts in large capacities,
whose last waves have no tokens: codes bit for bit, outputs against float64 attention."""
import numpy as np
import pytest

from oracle import aatc as ora

from helpers import rel_l2, stored_to_torch
from test_gpu_decode_runs import TOL, _decode, _reference, _setup

pytestmark = pytest.mark.gpu


def _check(lens, cap, append, **over):
    w, cal_k, cal_v, kc, ka, vc, va, q = args = _setup(2, lens, cap, **over)
    H, x = w.n_kv_heads, None
    if append:
        new = {t: np.stack([np.stack([w.cache(b, h, t, n=1)[0] for h in range(H)])
                            for b in range(len(lens))]) for t in "kv"}
        x = [stored_to_torch(new[t]) for t in "kv"]
    got, (kg, kag, vg, vag) = _decode(*args, lens, cap, x)
    ref = _reference(w, cal_k, cal_v, kg, kag, vg, vag, q, lens)
    for b, n in enumerate(lens):
        for h in range(H if append else 0):
            rec, a16, _ = ora.encode(w.as_f32(new["k"][b, h])[None], cal_k[h])
            np.testing.assert_array_equal(kg[b, h, n - 1].numpy(), rec[0])
            assert kag[b, h, n - 1].numpy().view(np.uint16) == a16.view(np.uint16)[0]
            rec, a16, _ = ora.encode(w.as_f32(new["v"][b, h])[None], cal_v[h])
            vrec = ora.tiles_to_records(vg[b, h].numpy(), cal_v[h].record_bytes)
            np.testing.assert_array_equal(vrec[n - 1], rec[0])
            assert vag[b, h, n - 1].numpy().view(np.uint16) == a16.view(np.uint16)[0]
        for j in range(got.shape[1]):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))


@pytest.mark.parametrize("runs", [1, 2, 3, 4, 5, 31, 32, 33])
def test_runs_of_512(runs):
    n = 512 * runs + 1                                # (the token itself is no part of a run)
    print(f"[append runs] {runs}", flush=True)
    _check([n], (n + 63) // 64 * 64, True, n_q_heads=4, n_kv_heads=1)


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("n", [1, 2, 128, 129, 513, 514, 1024, 1025, 1026, 2050])
def test_short_in_a_large_capacity(n, append):
    """1024-token chunks, one per workgroup: whole waves and the second half without tokens."""
    print(f"[short] {n} {append}", flush=True)
    _check([n], 32768, append, n_q_heads=16, n_kv_heads=8)


@pytest.mark.parametrize("n", [513, 1025, 1537, 2049])
def test_widest_records(n):
    """128-byte records: the most transfers per wave in flight, on two or three waves."""
    _check([n], (n + 63) // 64 * 64, True, avg_bits=8.0, b_max=16, n_q_heads=4, n_kv_heads=1)


def test_ragged_runs():
    _check([1, 1500, 4000, 64, 20000, 700, 513], 20032, True, n_q_heads=8, n_kv_heads=2)
    _check([5000, 300], 5056, True, avg_bits=6.0, b_max=12, n_q_heads=7, n_kv_heads=1)
