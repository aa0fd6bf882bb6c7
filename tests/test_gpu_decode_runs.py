"""GPU parity of the decode kernel's work split: runs of chunks per workgroup, runs dealt by
the lengths of a ragged batch, query heads in groups, records wider than 64 bytes, and the
fused append with few runs per row, against the oracle's float64 attention.

Caches hold random code bits and scales (a decode reads any bits); tolerance 2e-5 relative
L2 per query head: scores up to about 40 in the log2 domain rounded to 24 bits move a weight
by 2e-6 of itself, and the inverse transform in bf16 pairs adds about 2^-16 / 3.
"""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora

from helpers import device_params, rel_l2, stored_to_torch

pytestmark = pytest.mark.gpu
TOL = 2e-5


def _setup(cfg, lens, cap, avg_bits=2.75, b_max=8, scale=None, **overrides):
    w = workload(cfg, n_tokens=64, batch=len(lens), **overrides)
    H, B = w.n_kv_heads, len(lens)
    cal_k = [ora.calibrate(w.calib(h, "k"), avg_bits, b_max=b_max) for h in range(H)]
    cal_v = [ora.calibrate(w.calib(h, "v"), avg_bits, b_max=b_max) for h in range(H)]
    rk, rv = cal_k[0].record_bytes, cal_v[0].record_bytes
    g = torch.Generator().manual_seed(cfg * 1000 + cap)
    kc = torch.randint(0, 256, (B, H, cap, rk), dtype=torch.uint8, generator=g)
    vc = torch.randint(0, 256, (B, H, cap // 64, 64 * rv), dtype=torch.uint8, generator=g)
    ka = (0.2 + 0.8 * torch.rand((B, H, cap), generator=g))
    va = (0.5 + torch.rand((B, H, cap), generator=g))
    if scale is not None:                       # key scales by position
        ka = ka * scale
    ka, va = (t.to(torch.float16).view(torch.int16) for t in (ka, va))
    q = np.stack([w.queries(b) for b in range(B)])
    return w, cal_k, cal_v, kc, ka, vc, va, q


def _reference(w, cal_k, cal_v, kc, ka, vc, va, q, lens):
    H, G = w.n_kv_heads, w.n_q_heads // w.n_kv_heads
    out = np.zeros((len(lens), w.n_q_heads, 128))
    for b, n in enumerate(lens):
        if n == 0:
            continue
        q32 = w.as_f32(q[b])
        for h in range(H):
            k = ora.decode_tokens(kc[b, h, :n].numpy(), ka[b, h, :n].numpy().view(np.float16), cal_k[h])
            rec = ora.tiles_to_records(vc[b, h].numpy(), cal_v[h].record_bytes)[:n]
            v = ora.decode_tokens(rec, va[b, h, :n].numpy().view(np.float16), cal_v[h])
            out[b, h * G:(h + 1) * G] = ora.softmax_attention(q32[h * G:(h + 1) * G], k, v,
                                                              1 / np.sqrt(128))
    return out


def _decode(w, cal_k, cal_v, kc, ka, vc, va, q, lens, cap, x=None):
    B, H, HQ = len(lens), w.n_kv_heads, w.n_q_heads
    pk, pv = device_params(cal_k), device_params(cal_v)
    out = torch.full((B, HQ, 128), float("nan"), device="cuda")
    ws = torch.zeros(P.aatc_decode_workspace_bytes(B, HQ, H, cap), dtype=torch.uint8, device="cuda")
    lt = torch.tensor(lens, dtype=torch.int32, device="cuda")
    dev = [t.cuda() for t in (kc, ka, vc, va)]
    qt = stored_to_torch(q).cuda()
    tail = (lt, cap, cal_k[0].record_bytes, cal_v[0].record_bytes, 1 / np.sqrt(128), out, ws)
    for _ in range(2):                          # (the second call: counters left at zero)
        if x is None:
            P.aatc_decode_attention(pk, pv, B, HQ, H, qt, *dev, *tail)
        else:
            P.aatc_append_decode_attention(pk, pv, B, HQ, H, qt, x[0].cuda(), x[1].cuda(), *dev, *tail)
    torch.cuda.synchronize()
    return out.cpu().numpy(), [t.cpu() for t in dev]


CASES = {
    # more chunks than compute units: runs dealt by the lengths, an empty and a one-token row
    "ragged_runs": dict(cfg=2, lens=[11300, 5000, 1, 0, 1025], cap=11328),
    # the same, seven query heads per KV head, 512-token chunks (128-byte tile rows)
    "ragged_runs_gqa7_4bit": dict(cfg=3, lens=[9000, 513, 8704, 70, 1], cap=9024, avg_bits=4.0,
                                  n_kv_heads=8, n_q_heads=56),
    # more sequences than lanes of a wave
    "batch_70": dict(cfg=1, lens=[(37 * i) % 5000 for i in range(70)], cap=5056),
    # more rows than compute units
    "rows_320": dict(cfg=2, lens=[(411 * i) % 1100 for i in range(40)], cap=1152),
    # one sequence, equal runs of several chunks and a short last run; capacity far above it
    "one_sequence": dict(cfg=3, lens=[4999], cap=140000 // 64 * 64, n_kv_heads=2, n_q_heads=8),
    # query heads in two groups of eight, the second ragged
    "gqa12": dict(cfg=2, lens=[1500, 300], cap=1536, n_q_heads=24, n_kv_heads=2),
    "gqa16_runs": dict(cfg=2, lens=[9000] * 2, cap=9024, n_q_heads=128, n_kv_heads=8),
    # records of 80, 96, 112 and 128 bytes (the last two four query heads per workgroup), and
    # 144 (the general kernel)
    "bits5": dict(cfg=2, lens=[1030, 7], cap=1088, avg_bits=5.0),
    "bits6_gqa7": dict(cfg=3, lens=[1030, 512], cap=1088, avg_bits=6.0, b_max=12),
    "bits7_gqa7": dict(cfg=3, lens=[600, 1], cap=640, avg_bits=7.0, b_max=16),
    "bits8": dict(cfg=2, lens=[1030, 511], cap=1088, avg_bits=8.0, b_max=16),
    "bits9": dict(cfg=2, lens=[300], cap=320, avg_bits=9.0, b_max=16),
}


@pytest.mark.parametrize("name", list(CASES))
def test_decode_runs(name):
    print(f"[runs] {name}", flush=True)
    spec = CASES[name]
    args = _setup(**spec)
    got, _ = _decode(*args, spec["lens"], spec["cap"])
    ref = _reference(*args, spec["lens"])
    for b, n in enumerate(spec["lens"]):
        if n == 0:
            assert np.all(got[b] == 0)
        for j in range(got.shape[1] if n else 0):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))


@pytest.mark.parametrize("rising", [False, True])
def test_running_maximum_across_chunks(rising):
    """A run whose scores grow (or shrink) a hundredfold from chunk to chunk: the running
    maximum and the chunk exponents cover ranges far beyond 2^127."""
    cap = 8 * 1024
    pos = torch.arange(cap) // 1024
    scale = 0.01 * 2.2 ** (pos if rising else 7 - pos).float()
    args = _setup(2, [cap], cap, scale=scale, n_q_heads=1024, n_kv_heads=128)
    w = args[0]
    got, _ = _decode(*args, [cap], cap)
    ref = _reference(*args, [cap])
    err = [rel_l2(got[0, j], ref[0, j]) for j in range(w.n_q_heads)]
    # (scores up to about 200 in the log2 domain: rounding moves the weights by 2e-5)
    assert max(err) <= 10 * TOL, max(err)


@pytest.mark.parametrize("lens,cap,over", [
    ([1, 2, 777], 832, {}),                              # one or two runs per row
    ([4000], 4032, {}),                                  # eight
    ([11300, 64, 0, 5001], 11328, {}),                   # dealt by the lengths
    ([700, 65], 704, dict(n_q_heads=28, n_kv_heads=4)),
    ([520, 3], 576, dict(avg_bits=6.0, b_max=12)),       # wide records, fused
    ([520, 3], 576, dict(avg_bits=8.0, b_max=16, n_q_heads=56)),   # separate append
])
def test_append_with_few_runs(lens, cap, over):
    """The appended token's codes equal the oracle's encode and its term enters the output."""
    over = dict(over)
    args = _setup(2, lens, cap, over.pop("avg_bits", 2.75), over.pop("b_max", 8), **over)
    w, cal_k, cal_v, kc, ka, vc, va, q = args
    B, H = len(lens), w.n_kv_heads
    new = {t: np.stack([np.stack([w.cache(b, h, t, n=1)[0] for h in range(H)]) for b in range(B)])
           for t in "kv"}
    x = [stored_to_torch(new[t]) for t in "kv"]
    got, (kg, kag, vg, vag) = _decode(*args, lens, cap, x)
    for b, n in enumerate(lens):
        for h in range(H if n else 0):
            rec, a16, _ = ora.encode(w.as_f32(new["k"][b, h])[None], cal_k[h])
            np.testing.assert_array_equal(kg[b, h, n - 1].numpy(), rec[0])
            assert kag[b, h, n - 1].numpy().view(np.uint16) == a16.view(np.uint16)[0]
            rec, a16, _ = ora.encode(w.as_f32(new["v"][b, h])[None], cal_v[h])
            vrec = ora.tiles_to_records(vg[b, h].numpy(), cal_v[h].record_bytes)
            np.testing.assert_array_equal(vrec[n - 1], rec[0])
            assert vag[b, h, n - 1].numpy().view(np.uint16) == a16.view(np.uint16)[0]
            old = ora.tiles_to_records(vc[b, h].numpy(), cal_v[h].record_bytes)
            np.testing.assert_array_equal(vrec[:n - 1], old[:n - 1])
            np.testing.assert_array_equal(kg[b, h, :n - 1].numpy(), kc[b, h, :n - 1].numpy())
    ref = _reference(w, cal_k, cal_v, kg, kag, vg, vag, q, lens)
    for b, n in enumerate(lens):
        for j in range(got.shape[1] if n else 0):
            assert rel_l2(got[b, j], ref[b, j]) <= TOL, (b, n, j, rel_l2(got[b, j], ref[b, j]))
