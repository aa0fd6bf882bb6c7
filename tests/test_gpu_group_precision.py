"""Precision of the head-group decode at 16 to 32 query heads per group, whose matrix-core products
take query weights and probabilities as sums of two fp16 numbers (22 bits), against float64
attention over the stored codes; and NaN and infinite queries there.

Bar 2e-5 relative L2 per head: the terms of a score add up to about 40 in magnitude (log2 domain),
each within 2^-22 of itself, so a score moves by under 1e-5 and a weight by 0.7 of that; the
probabilities add 2^-22, the fp32 sums and the hardware exp2 about as much again (2 to 8e-6 in all
measured).  One fp16 number instead of two (11 bits) is 2^11 times as far off per term: the same
queries rounded so on the reference's side miss the bar."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from oracle import aatc as ora

from helpers import group_device_params, rel_l2
from test_gpu_groups import GCase, _run

pytestmark = pytest.mark.gpu
TOL = 2e-5


def _case(gkv, heads, quantizer, lens):
    case = GCase(2, gkv, lens, quantizer=quantizer, n_kv_heads=gkv, n_q_heads=heads)
    pk, pv = group_device_params(case.cal["k"]), group_device_params(case.cal["v"])
    cache = [*case.gpu_encode(pk, "k"), *case.gpu_encode(pv, "v")]

    def decode(q):
        B = len(lens)
        out = torch.full((B, heads, 128), 7.0, device="cuda")
        ws = torch.empty(P.aatc_group_decode_workspace_bytes(B, heads, gkv, gkv, case.cap),
                         dtype=torch.uint8, device="cuda")
        P.aatc_group_decode_attention(pk, pv, B, heads, gkv, gkv, torch.from_numpy(q).cuda(), *cache,
                                      torch.tensor(lens, dtype=torch.int32, device="cuda"), case.cap,
                                      case.R["k"], case.R["v"], 128 ** -0.5, out, ws)
        torch.cuda.synchronize()
        return out.cpu().numpy()
    q = case.w.as_f32(case.queries()).astype(np.float32)
    return case, cache, q, decode


def _weights(q, cal, block):
    """The log2-domain weight per unit of code and token scale of every channel."""
    qt = q.astype(np.float64) @ cal.T32[128 * block:128 * block + 128].astype(np.float64)
    step = np.where(cal.bits > 0, cal.s16.astype(np.float64) * np.exp2(1.0 - cal.bits), 0.0)
    return qt * step * (128 ** -0.5 * np.log2(np.e))


def _attend(w, level, alpha, v):
    z = (level @ w) * alpha
    p = np.exp2(z - z.max())
    return (p / p.sum()) @ v


@pytest.mark.timeout(300)
@pytest.mark.parametrize("quantizer", ["midtread", "midrise"])
@pytest.mark.parametrize("gkv,heads", [(4, 16), (1, 17), (4, 28), (2, 32)])
def test_against_float64(gkv, heads, quantizer):
    print(f"[group precision] {gkv} {heads} {quantizer}", flush=True)
    lens = [1500, 300]
    case, (kc, ka, vc, va), q, decode = _case(gkv, heads, quantizer, lens)
    ck, cv = case.cal["k"][0], case.cal["v"][0]
    got, rounded = decode(q), []
    for b, n in enumerate(lens):
        rec = kc[b, 0, :n].cpu().numpy()
        level = ora.unpack_records(rec, ck.bits) + (0.5 if quantizer == "midrise" else 0.0)
        alpha = ka[b, 0, :n].cpu().numpy().view(np.float16).astype(np.float64)
        v = ora.decode_tokens(vc[b, 0, :n].cpu().numpy(), va[b, 0, :n].cpu().numpy().view(np.float16), cv)
        for j in range(heads):
            kk = j // (heads // gkv)
            w = _weights(q[b, j], ck, kk)
            vb = v[:, 128 * kk:128 * kk + 128]
            ref = _attend(w, level, alpha, vb)
            err = rel_l2(got[b, j], ref)
            assert err <= TOL, (b, j, err)
            s = np.exp2(np.floor(np.log2(np.abs(w).max())) - 14)     # the kernel's scaling
            rounded.append(rel_l2(_attend((w / s).astype(np.float16).astype(np.float64) * s, level, alpha, vb), ref))
    assert np.median(rounded) > 2 * TOL                              # one fp16 number would miss the bar


@pytest.mark.timeout(300)
@pytest.mark.parametrize("gkv,heads", [(4, 16), (1, 17), (2, 32)])
def test_nan_queries(gkv, heads):
    """NaN in their heads, the very same bits in the others, zeros for an empty sequence."""
    lens = [600, 0, 1]
    _, _, q, decode = _case(gkv, heads, "midtread", lens)
    good = decode(q)
    bad = {1: np.nan, heads - 1: np.inf}
    for j, v in bad.items():
        q[:, j, 5] = v
    got = decode(q)
    for b, n in enumerate(lens):
        for j in range(heads):
            if n == 0:
                assert np.all(got[b, j] == 0)
            elif j in bad:
                assert np.all(np.isnan(got[b, j])), (b, j, got[b, j, :4])
            else:
                np.testing.assert_array_equal(got[b, j], good[b, j])


@pytest.mark.parametrize("gkv,heads", [(1, 16), (2, 20), (1, 32)])
def test_codes_over_12_bits(gkv, heads):
    """fp16 does not hold them: the VALU body inside the matrix-core launch."""
    lens = [700, 0, 257]
    case = GCase(2, gkv, lens, avg_bits=8.0, b_max=16, n_kv_heads=gkv, n_q_heads=heads)
    assert max(c.bits.max() for t in "kv" for c in case.cal[t]) > 12
    _run(case)
