"""GPU parity of the decode and of the append step with key and value records of different sizes,
values wider than keys among them (fewer heads or tokens per workgroup), against the oracle's
float64 attention; tolerance and caches of random bits as in test_gpu_decode_runs."""
import numpy as np
import pytest
import torch

from oracle import aatc as ora

from helpers import rel_l2, stored_to_torch
from test_gpu_decode_runs import TOL, _decode, _reference, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("rk,rv,hq,hkv,lens,cap", [
    (64, 96, 14, 2, [700, 33], 704),                    # Qwen's group at 4-bit keys, 6-bit values
    (36, 96, 10, 2, [513, 1], 576),
    (92, 96, 24, 2, [600, 0], 640),                     # more heads than one workgroup
    (12, 128, 16, 2, [300, 70], 320),                   # four heads
    (128, 20, 4, 2, [530], 576),
    (24, 64, 96, 8, [900, 130, 1, 64, 65, 10, 520, 300], 2048)])   # 1024-token chunks do not fit
def test_record_pairs(rk, rv, hq, hkv, lens, cap, append):
    print(f"[pairs] {rk} {rv} {hq}/{hkv} append {append}", flush=True)
    over = dict(n_q_heads=hq, n_kv_heads=hkv, b_max=12)
    w, cal_k, _, kc, ka, _, _, q = _setup(2, lens, cap, avg_bits=rk / 16, **over)
    _, _, cal_v, _, _, vc, va, _ = _setup(2, lens, cap, avg_bits=rv / 16, **over)
    assert (cal_k[0].record_bytes, cal_v[0].record_bytes) == (rk, rv)
    new = {t: np.stack([np.stack([w.cache(b, h, t, n=1)[0] for h in range(hkv)])
                        for b in range(len(lens))]) for t in "kv"}
    x = [stored_to_torch(new[t]) for t in "kv"] if append else None
    got, (kg, kag, vg, vag) = _decode(w, cal_k, cal_v, kc, ka, vc, va, q, lens, cap, x)
    for b, n in enumerate(lens):
        for h in range(hkv if n and append else 0):
            rec, a16, _ = ora.encode(w.as_f32(new["k"][b, h])[None], cal_k[h])
            np.testing.assert_array_equal(kg[b, h, n - 1].numpy(), rec[0])
            rec, a16, _ = ora.encode(w.as_f32(new["v"][b, h])[None], cal_v[h])
            np.testing.assert_array_equal(ora.tiles_to_records(vg[b, h].numpy(), rv)[n - 1], rec[0])
            assert vag[b, h, n - 1].numpy().view(np.uint16) == a16.view(np.uint16)[0]
    ref = _reference(w, cal_k, cal_v, kg, kag, vg, vag, q, lens)
    for b, n in enumerate(lens):
        assert n or np.all(got[b] == 0)
        for j in range(hq if n else 0):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))
