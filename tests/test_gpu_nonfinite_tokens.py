"""Tokens with NaN or infinite elements, and tokens far above 1, on every encode route: the codes
and scale of the exact routine, which takes a NaN's or an infinity's bits as the number they spell
at exponent 255 (so the scale saturates), whatever the kernel, and nothing else changes."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora
from oracle import groups as og

from helpers import (alpha_cache, device_params, group_device_params, record_cache, stored_to_torch,
                     tile_cache)
from test_gpu_decode_runs import _setup

pytestmark = pytest.mark.gpu


def _rows(x):
    """Six rows of x [n >= 6, d] replaced; their indices."""
    n, d = x.shape
    at = np.linspace(0, n - 1, 6).astype(int)
    x[at[0], 1] = np.inf
    x[at[1], d - 1] = -np.inf
    x[at[2], d // 2] = np.nan
    x[at[3]] = np.nan
    x[at[4]] = np.float32(2.0 ** 127)
    # one element of 2^43, the others below what 22 bits beside it hold, one subnormal
    x[at[5]] = np.float32(2.0 ** 19)
    x[at[5], 0], x[at[5], 3] = np.float32(2.0 ** 43), np.float32(2.0 ** -133)
    return at


def _spelled(x32):
    """The numbers of fp32 bit patterns, exponent 255 read like any other (float64)."""
    b = np.ascontiguousarray(x32, np.float32).view(np.uint32)
    ef, m = (b >> 23) & 255, b & 0x7FFFFF
    v = np.where(ef > 0, m | 0x800000, m) * np.exp2(np.where(ef > 0, ef, 1) - 150.0)
    return np.where(b >> 31, -v, v)


def _encode(x32, cal):
    """(records, scale bits) of rows x32, h from the definition in rational arithmetic."""
    xs = _spelled(x32)
    h = np.array([[ora.exact_dot_f32(r, cal.T32[:, c]) if cal.bits[c] else np.float32(0)
                   for c in range(cal.T32.shape[1])] for r in xs], dtype=np.float32)
    bits = cal.bits.astype(np.int64)
    inv_s = ora.inverse_f32(cal.s16.astype(np.float32))
    with np.errstate(over="ignore", invalid="ignore"):
        r = np.where(bits > 0, h * inv_s, np.float32(0)).astype(np.float32)
        a16 = np.minimum(np.abs(r).max(axis=1), np.float32(65504)).astype(np.float16)
        xq = (r * ora.inverse_f32(a16.astype(np.float32))[:, None]).astype(np.float32).astype(np.float64)
        xq = np.clip(xq * np.exp2(np.maximum(bits - 1, 0)), -2.0 ** 20, 2.0 ** 20)
    code = np.floor(xq) if cal.quantizer == "midrise" else np.floor(xq + 0.5)   # (exact in fp64)
    half = 1 << np.maximum(bits - 1, 0)
    code = np.clip(code.astype(np.int64), np.where(bits > 0, -half, 0), np.where(bits > 0, half - 1, 0))
    return ora.pack_records(code, cal.bits), a16.view(np.uint16)


def _tokens(n, heads, dtype):
    g = torch.Generator().manual_seed(n)
    x = (4 * torch.randn((n, heads, 128), generator=g)).to(
        torch.bfloat16 if dtype == "bf16" else torch.float32).float().numpy()
    return x


@pytest.mark.parametrize("quantizer", ["midtread", "midrise"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,odd", [(7, 0), (100, 0), (100, 1)])     # each of the three kernels
def test_encode(n, odd, dtype, quantizer):
    print(f"[nonfinite] {n} {odd} {dtype} {quantizer}", flush=True)
    H = 2
    w = workload(2, n_tokens=64, n_kv_heads=H, n_q_heads=H)
    cal = [ora.calibrate(w.calib(h, "k"), 2.75) for h in range(H)]
    for c in cal:
        c.quantizer = quantizer
    x = _tokens(n, H, dtype)
    at = _rows(x[:, 0])
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    xt = torch.zeros((n, H * 128 + odd), dtype=td)
    xt[:, :H * 128] = torch.from_numpy(x.reshape(n, H * 128)).to(td)
    xg, params, cap, rb = xt.cuda(), device_params(cal), (n + 63) // 64 * 64, cal[0].record_bytes
    kc, vc = record_cache(H, cap, rb), tile_cache(H, cap, rb)
    ka, va = alpha_cache(H, cap), alpha_cache(H, cap)
    P.aatc_encode(params, H, xg, n, H * 128 + odd, P.LAYOUT_RECORDS, kc, ka, cap, 0)
    P.aatc_encode(params, H, xg, n, H * 128 + odd, P.LAYOUT_TILES, vc, va, cap, 0)
    torch.cuda.synchronize()
    xs = xt[:, :H * 128].float().numpy().reshape(n, H, 128)
    for h in range(H):
        want = np.zeros((n, rb), np.uint8), np.zeros(n, np.uint16)
        plain = np.setdiff1d(np.arange(n), at) if h == 0 else np.arange(n)
        rec, a16, _ = ora.encode(xs[plain, h], cal[h])
        want[0][plain], want[1][plain] = rec, a16.view(np.uint16)
        if h == 0:
            want[0][at], want[1][at] = _encode(xs[at, h], cal[h])
        np.testing.assert_array_equal(kc[h, :n].cpu().numpy(), want[0])
        np.testing.assert_array_equal(ora.tiles_to_records(vc[h].cpu().numpy(), rb)[:n], want[0])
        for a in (ka, va):
            np.testing.assert_array_equal(a[h, :n].cpu().numpy().view(np.uint16), want[1])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("gkv,n", [(1, 3000), (2, 40)])
def test_group_encode(gkv, n, dtype):
    print(f"[nonfinite group] {gkv} {n} {dtype}", flush=True)
    d = 128 * gkv
    w = workload(2, n_tokens=64, n_kv_heads=gkv, n_q_heads=gkv)
    cal = og.calibrate_group(np.concatenate([w.calib(h, "k") for h in range(gkv)], axis=1), 2.75, b_max=8)
    x = _tokens(n, gkv, dtype).reshape(n, d)
    at = _rows(x)
    xt = torch.from_numpy(x).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    xs = xt.float().numpy()
    codes, al = record_cache(1, n, cal.record_bytes), alpha_cache(1, n)
    P.aatc_group_encode(group_device_params([cal]), 1, gkv, xt.cuda(), n, d, codes, al, n, 0)
    torch.cuda.synchronize()
    want = np.zeros((n, cal.record_bytes), np.uint8), np.zeros(n, np.uint16)
    plain = np.setdiff1d(np.arange(n), at)
    rec, a16, _ = og.encode_group(xs[plain], cal)
    want[0][plain], want[1][plain] = rec, a16.view(np.uint16)
    want[0][at], want[1][at] = _encode(xs[at], cal)
    np.testing.assert_array_equal(codes[0].cpu().numpy(), want[0])
    np.testing.assert_array_equal(al[0].cpu().numpy().view(np.uint16), want[1])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_tok,bits,b_max", [(65, 2.75, 8), (65, 6.0, 12), (65, 8.0, 12), (12000, 2.75, 8)])
def test_append(n_tok, bits, b_max, dtype):
    """Appended in one launch with the decode: few runs per row, and more than 32."""
    print(f"[nonfinite append] {n_tok} {bits} {dtype}", flush=True)
    B, H, HQ = 6, 1, 4
    lens, cap = [n_tok] + [65] * (B - 1), (n_tok + 63) // 64 * 64
    w, cal_k, cal_v, kc, ka, vc, va, q = _setup(2, lens, cap, avg_bits=bits, b_max=b_max, n_q_heads=HQ,
                                                n_kv_heads=H)
    x = _tokens(B, 1, dtype)[:, 0]
    at = _rows(x)
    assert sorted(at) == list(range(B))
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    xt = torch.from_numpy(x).to(td)
    xs = xt.float().numpy()
    dev = [t.cuda() for t in (kc, ka, vc, va)]
    out = torch.zeros((B, HQ, 128), device="cuda")
    ws = torch.zeros(P.aatc_decode_workspace_bytes(B, HQ, H, cap), dtype=torch.uint8, device="cuda")
    P.aatc_append_decode_attention(
        device_params(cal_k), device_params(cal_v), B, HQ, H, stored_to_torch(q).cuda(),
        xt.view(B, H, 128).cuda(), xt.view(B, H, 128).cuda(), *dev,
        torch.tensor(lens, dtype=torch.int32, device="cuda"), cap, cal_k[0].record_bytes,
        cal_v[0].record_bytes, 128 ** -0.5, out, ws)
    torch.cuda.synchronize()
    (krec, ka16), (vrec, va16) = _encode(xs, cal_k[0]), _encode(xs, cal_v[0])
    for b, n in enumerate(lens):
        np.testing.assert_array_equal(dev[0][b, 0, n - 1].cpu().numpy(), krec[b])
        got = ora.tiles_to_records(dev[2][b, 0].cpu().numpy(), cal_v[0].record_bytes)
        np.testing.assert_array_equal(got[n - 1], vrec[b])
        assert dev[1][b, 0, n - 1].cpu().numpy().view(np.uint16) == ka16[b]
        assert dev[3][b, 0, n - 1].cpu().numpy().view(np.uint16) == va16[b]
