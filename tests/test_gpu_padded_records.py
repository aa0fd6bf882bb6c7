"""Encode into records padded to another head's size (aatc_calibrate_bits, up to 256 bytes): the
record's bits and scales as without the padding, zeros behind them, nothing beyond the record."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora

from helpers import abi_calibration, alpha_cache, device_params, record_cache, tile_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("record", [48, 128, 132, 256])
@pytest.mark.parametrize("n,pos", [(5, 60), (100, 31), (700, 0)])
def test_padded_records(n, pos, record, dtype):
    print(f"[padded] {n} {pos} {record} {dtype}", flush=True)
    H = 2
    w = workload(2, n_tokens=n, n_kv_heads=H, n_q_heads=H, dtype=dtype)
    cal = [ora.calibrate(w.calib(h, "k"), 2.75) for h in range(H)]
    abi = [abi_calibration(c) for c in cal]
    for c in abi:
        c.record_bytes = record
    params, cap = device_params(abi), (pos + n + 63) // 64 * 64
    x = np.stack([w.as_f32(w.cache(0, h, "k")) for h in range(H)], axis=1)
    xt = torch.from_numpy(x).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    kc, vc = record_cache(H, cap, record).fill_(0xA5), tile_cache(H, cap, record)
    ka, va = alpha_cache(H, cap), alpha_cache(H, cap)
    P.aatc_encode(params, H, xt, n, H * 128, P.LAYOUT_RECORDS, kc, ka, cap, pos)
    P.aatc_encode(params, H, xt, n, H * 128, P.LAYOUT_TILES, vc, va, cap, pos)
    torch.cuda.synchronize()
    for h in range(H):
        rec, a16, _ = ora.encode(x[:, h], cal[h])
        want = np.zeros((n, record), np.uint8)
        want[:, :rec.shape[1]] = rec
        got = kc[h].cpu().numpy()
        np.testing.assert_array_equal(got[pos:pos + n], want)
        assert np.all(got[:pos] == 0xA5) and np.all(got[pos + n:] == 0xA5)
        np.testing.assert_array_equal(ora.tiles_to_records(vc[h].cpu().numpy(), record)[pos:pos + n], want)
        for a in (ka, va):
            np.testing.assert_array_equal(a[h, pos:pos + n].cpu().numpy().view(np.uint16),
                                          a16.view(np.uint16))
