"""Decode and append of batches past the sizes where the deal of the work changes: more than 512
sequences (whose lengths no longer fit the registers that hold the first), and rows of several
rounds of the chip, one run each whatever their lengths."""
import numpy as np
import pytest
import torch

from helpers import rel_l2
from test_gpu_decode_runs import TOL, _decode, _reference, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("batch,hkv,hq,cap", [
    (513, 1, 3, 1088),          # dealt by the lengths, the last sequence past the registers
    (600, 1, 8, 2112),          # runs of several chunks among them
    (130, 8, 16, 1088)])        # 1040 rows of at most two chunks: one run each
def test_large_batches(batch, hkv, hq, cap, append):
    print(f"[large] {batch} {hkv} {hq} {cap} {append}", flush=True)
    lens = [(97 * i) % 150 for i in range(batch)]
    for i in (0, 63, 64, batch // 2, batch - 2, batch - 1):
        lens[i] = cap - i % 3
    lens[1], lens[batch - 3] = 1025, 1024
    w, cal_k, cal_v, kc, ka, vc, va, q = args = _setup(2, lens, cap, n_kv_heads=hkv, n_q_heads=hq)
    x = None
    if append:
        g = torch.Generator().manual_seed(4)
        x = [torch.randn((batch, hkv, 128), generator=g) for _ in range(2)]
    got, (kg, kag, vg, vag) = _decode(*args, lens, cap, x)
    # every long sequence and a share of the short ones against the oracle, all rows for the rest
    check = sorted({*[i for i, n in enumerate(lens) if n > 150], *range(5, batch, 17)})
    sub = [lens[i] if i in check else 0 for i in range(batch)]
    ref = _reference(w, cal_k, cal_v, kg, kag, vg, vag, q, sub)
    for b, n in enumerate(lens):
        assert np.all(np.isfinite(got[b])) and (n > 0 or np.all(got[b] == 0)), b
        for j in range(hq if sub[b] else 0):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))
