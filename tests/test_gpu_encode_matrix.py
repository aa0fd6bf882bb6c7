"""GPU parity of the matrix-core encodes at the sizes and values where they can go wrong,
bit for bit against the oracle: fp32 tokens (four limbs) of both layouts and readings, head
groups at every tile height and channel count, rows that are not 16-byte aligned, and tokens
whose certificate fails (the exact kernels redo them)."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora
from oracle import groups as og

from helpers import (alpha_cache, device_params, group_device_params, record_cache,
                     stored_to_torch, tile_cache)

pytestmark = pytest.mark.gpu


def _hard_tokens(x, seed):
    """Some rows of x [n, d] replaced by values the fixed-point form finds hard."""
    rng = np.random.default_rng(seed)
    n, d = x.shape
    rows = rng.permutation(n)[:8] if n >= 16 else np.arange(min(n, 8))
    edge = [lambda r: np.zeros_like(r),                               # a zero token
            lambda r: np.round(r * 4) / 4,                            # ties
            lambda r: r * np.float32(2.0) ** rng.integers(-20, 1, d), # 20 binades
            lambda r: r * np.float32(2.0 ** -60),                     # far below 1
            lambda r: r * np.float32(2.0 ** 30),                      # a saturating scale
            lambda r: r * np.float32(2.0) ** rng.integers(-60, 1, d), # 60 binades
            lambda r: np.where(np.arange(d) == 3, r, np.float32(0)),  # one element
            lambda r: r * np.float32(2.0 ** -140)]                    # subnormals
    x = x.copy()
    for i, f in zip(rows, edge):
        x[i] = f(x[i]).astype(np.float32)
    return x


@pytest.mark.parametrize("n,pos,avg,quantizer", [
    (17, 0, 2.75, "midtread"), (63, 1, 4.0, "midrise"), (129, 31, 2.0, "midrise"),
    (500, 65, 4.0, "midtread"), (1500, 7, 2.75, "midtread")])
def test_f32_tokens(n, pos, avg, quantizer):
    print(f"[f32] {n} {pos} {avg} {quantizer}", flush=True)
    H = 3
    w = workload(5, n_tokens=n, n_kv_heads=H, n_q_heads=H, dtype="f32")
    cal = [ora.calibrate(w.calib(h, "k"), avg, q_calib=w.calib_queries(h), group=w.group)
           for h in range(H)]                       # (query-weighted: dropped channels at 2 bits)
    for c in cal:
        c.quantizer = quantizer
    x = np.stack([_hard_tokens(w.cache(0, h, "k"), h) for h in range(H)], axis=1)
    params, cap, rb = device_params(cal), (pos + n + 63) // 64 * 64, cal[0].record_bytes
    xt = torch.from_numpy(x).cuda()
    kc, vc = record_cache(H, cap, rb).fill_(0xA5), tile_cache(H, cap, rb)
    ka, va = alpha_cache(H, cap), alpha_cache(H, cap)
    P.aatc_encode(params, H, xt, n, H * 128, P.LAYOUT_RECORDS, kc, ka, cap, pos)
    P.aatc_encode(params, H, xt, n, H * 128, P.LAYOUT_TILES, vc, va, cap, pos)
    torch.cuda.synchronize()
    for h in range(H):
        rec, a16, _ = ora.encode(x[:, h], cal[h])
        got = kc[h].cpu().numpy()
        bad = np.argwhere(np.any(got[pos:pos + n] != rec, axis=1)).ravel()
        assert bad.size == 0, (h, bad[:5])
        assert np.all(got[:pos] == 0xA5) and np.all(got[pos + n:] == 0xA5)
        np.testing.assert_array_equal(ora.tiles_to_records(vc[h].cpu().numpy(), rb)[pos:pos + n], rec)
        for a in (ka, va):
            np.testing.assert_array_equal(a[h, pos:pos + n].cpu().numpy().view(np.uint16),
                                          a16.view(np.uint16))


@pytest.mark.parametrize("gkv,groups,n,dtype,quantizer,odd", [
    (4, 1, 1, "bf16", "midtread", 0), (4, 2, 33, "f32", "midrise", 0),      # 16 tokens a workgroup
    (4, 8, 784, "bf16", "midrise", 0), (4, 8, 1552, "bf16", "midtread", 0), # 32, 64
    (4, 8, 800, "f32", "midtread", 0),                                      # 32
    (3, 8, 1553, "bf16", "midtread", 0), (3, 1, 70, "f32", "midtread", 1),
    (2, 8, 1601, "bf16", "midrise", 1), (1, 8, 1555, "bf16", "midtread", 0),
    (1, 2, 100, "f32", "midtread", 1)])
def test_group_tokens(gkv, groups, n, dtype, quantizer, odd):
    print(f"[group] {gkv} {groups} {n} {dtype} {quantizer} {odd}", flush=True)
    H, d = gkv * groups, 128 * gkv
    w = workload(2, n_tokens=n, n_kv_heads=H, n_q_heads=H, dtype=dtype)
    check = [0, groups - 1]
    cals = {g: og.calibrate_group(np.concatenate(
        [w.calib(h, "k") for h in range(g * gkv, (g + 1) * gkv)], axis=1), 2.75, b_max=8,
        quantizer=quantizer) for g in set(check)}
    cal = [cals.get(g, cals[0]) for g in range(groups)]
    stored = np.stack([w.cache(0, h, "k") for h in range(H)], axis=1).reshape(n, H * 128)
    if dtype == "f32":
        for g in check:
            stored[:, g * d:(g + 1) * d] = _hard_tokens(stored[:, g * d:(g + 1) * d], g)
    pos, cap = 5, n + 11
    xt = torch.zeros((n, H * 128 + odd), dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    xt[:, :H * 128] = stored_to_torch(stored)
    codes = record_cache(groups, cap, cal[0].record_bytes).fill_(0x5A)
    al = alpha_cache(groups, cap)
    P.aatc_group_encode(group_device_params(cal), groups, gkv, xt.cuda(), n, H * 128 + odd, codes,
                        al, cap, pos)
    torch.cuda.synchronize()
    x32 = w.as_f32(stored)
    for g in check:
        rec, a16, _ = og.encode_group(x32[:, g * d:(g + 1) * d], cals[g])
        got = codes[g].cpu().numpy()
        bad = np.argwhere(np.any(got[pos:pos + n] != rec, axis=1)).ravel()
        assert bad.size == 0, (g, bad[:5])
        assert np.all(got[:pos] == 0x5A) and np.all(got[pos + n:] == 0x5A)
        np.testing.assert_array_equal(al[g, pos:pos + n].cpu().numpy().view(np.uint16),
                                      a16.view(np.uint16))
