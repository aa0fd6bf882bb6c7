"""Decode and append of more rows than compute units, one chunk of capacity each: dealt without the
lengths, in more than one round of the chip, empty and one-token rows among them."""
import numpy as np
import pytest
import torch

from oracle import aatc as ora

from helpers import rel_l2
from test_gpu_decode_runs import TOL, _decode, _reference, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("cap,over", [(1024, {}), (512, dict(avg_bits=6.0, b_max=12)),
                                      (448, dict(n_q_heads=96, n_kv_heads=8))])
def test_one_chunk_rows(cap, over, append):
    print(f"[one chunk] {cap} {over} {append}", flush=True)
    over, lens = dict(over), [(409 * i) % (cap + 1) for i in range(36)]
    lens[5], lens[6] = 1, cap
    args = _setup(2, lens, cap, over.pop("avg_bits", 2.75), over.pop("b_max", 8), **over)
    w, cal_k, cal_v, kc, ka, vc, va, q = args
    assert len(lens) * w.n_kv_heads > 256
    x = None
    if append:
        g = torch.Generator().manual_seed(3)
        x = [torch.randn((len(lens), w.n_kv_heads, 128), generator=g) for _ in range(2)]
    got, (kg, kag, vg, vag) = _decode(*args, lens, cap, x)
    ref = _reference(w, cal_k, cal_v, kg, kag, vg, vag, q, lens)
    for b, n in enumerate(lens):
        if n == 0:
            assert np.all(got[b] == 0)
            continue
        if append:
            rec, a16, _ = ora.encode(x[0][b, :1].numpy(), cal_k[0])
            np.testing.assert_array_equal(kg[b, 0, n - 1].numpy(), rec[0])
        for j in range(got.shape[1]):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))
