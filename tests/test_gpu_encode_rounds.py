"""The bulk encode of bf16 tokens on both of its workgroup sizes (eight waves, or twelve where eight
would take a round more), at the sizes where the choice changes: bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora

from helpers import alpha_cache, device_params, record_cache, stored_to_torch, tile_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quantizer", ["midtread", "midrise"])
@pytest.mark.parametrize("n,pos", [
    (1024, 0), (1024, 1),          # 64 heads, four workgroups each: 32 units, and 34 (twelve waves)
    (1505, 31), (1536, 0),         # the last sizes of one round of twelve
    (1537, 0), (3000, 5)])         # two rounds of each; three and two
def test_bf16_rounds(n, pos, quantizer):
    print(f"[rounds] {n} {pos} {quantizer}", flush=True)
    H, check = 64, [0, 63]
    w = workload(2, n_tokens=n, n_kv_heads=2, n_q_heads=2)
    two = [ora.calibrate(w.calib(h, "k"), 2.75) for h in range(2)]
    for c in two:
        c.quantizer = quantizer
    rows = [w.cache(0, h, "k") for h in range(2)]
    rng = np.random.default_rng(n)
    for r in rows:                                  # zeros, and elements far below the largest
        r[rng.integers(0, n, 4)] = 0
        small = rng.integers(0, n, 40)
        r[small, rng.integers(0, 128, 40)] = rng.integers(0x2000, 0x3000, 40).astype(np.uint16)
    x = torch.stack([stored_to_torch(rows[h % 2]) for h in range(H)], dim=1).contiguous()
    params = device_params([two[h % 2] for h in range(H)])
    cap, rb = (pos + n + 63) // 64 * 64, two[0].record_bytes
    kc, vc = record_cache(H, cap, rb).fill_(0xA5), tile_cache(H, cap, rb)
    ka, va = alpha_cache(H, cap), alpha_cache(H, cap)
    xg = x.cuda()
    P.aatc_encode(params, H, xg, n, H * 128, P.LAYOUT_RECORDS, kc, ka, cap, pos)
    P.aatc_encode(params, H, xg, n, H * 128, P.LAYOUT_TILES, vc, va, cap, pos)
    torch.cuda.synchronize()
    for h in check:
        rec, a16, _ = ora.encode(w.as_f32(rows[h % 2]), two[h % 2])
        got = kc[h].cpu().numpy()
        np.testing.assert_array_equal(got[pos:pos + n], rec)
        assert np.all(got[:pos] == 0xA5) and np.all(got[pos + n:] == 0xA5)
        np.testing.assert_array_equal(ora.tiles_to_records(vc[h].cpu().numpy(), rb)[pos:pos + n], rec)
        for a in (ka, va):
            np.testing.assert_array_equal(a[h, pos:pos + n].cpu().numpy().view(np.uint16),
                                          a16.view(np.uint16))
    for h in range(2, H):                           # the other heads repeat the first two
        assert torch.equal(kc[h], kc[h % 2]) and torch.equal(vc[h], vc[h % 2]) and torch.equal(ka[h], ka[h % 2])
