"""NaN and infinite queries: the outputs of their heads are NaN, not the zeros of an empty row, and
the other heads keep the very bits they have without them, on every form of the matrix-core decode
(head slots, records, append, segment) and on the general kernel."""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P

from helpers import device_params, stored_to_torch
from test_gpu_decode_runs import _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["plain", "append", "segment"])
@pytest.mark.parametrize("hq,hkv,bits,b_max", [
    (8, 2, 2.75, 8), (24, 2, 2.75, 8), (14, 2, 6.0, 12), (8, 2, 8.0, 12), (8, 2, 9.0, 16)])
def test_nan_queries(hq, hkv, bits, b_max, mode):
    print(f"[nan] {hq}/{hkv} {bits} {mode}", flush=True)
    lens, cap = [1500, 0, 1, 66], 1536
    w, cal_k, cal_v, kc, ka, vc, va, q = _setup(2, lens, cap, avg_bits=bits, b_max=b_max, n_q_heads=hq,
                                                n_kv_heads=hkv)
    B, R = len(lens), (cal_k[0].record_bytes, cal_v[0].record_bytes)
    pk, pv = device_params(cal_k), device_params(cal_v)
    lt = torch.tensor(lens, dtype=torch.int32, device="cuda")
    g = torch.Generator().manual_seed(1)
    x = [torch.randn((B, hkv, 128), generator=g).cuda() for _ in range(2)]
    seg = [torch.randn((B, hkv, 8, 128), generator=g).cuda() for _ in range(2)]
    n_seg = [3, 0, 0, 8]

    def run(qt):
        out = torch.full((B, hq, 128), 7.0, device="cuda")
        ws = torch.zeros(P.aatc_decode_workspace_bytes(B, hq, hkv, cap), dtype=torch.uint8, device="cuda")
        c = [t.cuda() for t in (kc, ka, vc, va)]
        tail = (lt, cap, *R, 128 ** -0.5)
        if mode == "append":
            P.aatc_append_decode_attention(pk, pv, B, hq, hkv, qt, *x, *c, *tail, out, ws)
        elif mode == "segment":
            P.aatc_decode_attention_segmented(pk, pv, B, hq, hkv, qt, *c, *tail, *seg,
                                              torch.tensor(n_seg, dtype=torch.int32, device="cuda"), 8,
                                              out, ws)
        else:
            P.aatc_decode_attention(pk, pv, B, hq, hkv, qt, *c, *tail, out, ws)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    qt = stored_to_torch(q).cuda()
    good = run(qt)
    bad_heads = {1: float("nan"), hq - 1: float("inf")}
    for j, v in bad_heads.items():
        qt[:, j, 5] = v
    got = run(qt)
    for b, n in enumerate(lens):
        empty = n == 0 and (mode != "segment" or n_seg[b] == 0)
        for j in range(hq):
            if empty:
                assert np.all(got[b, j] == 0), (b, j)
            elif j in bad_heads:
                assert np.all(np.isnan(got[b, j])), (b, j, got[b, j, :4])
            else:
                np.testing.assert_array_equal(got[b, j], good[b, j], err_msg=str((b, j)))


@pytest.mark.parametrize("hq", [8, 24])
def test_nan_query_on_a_segment_alone(hq):
    """No compressed token yet: the segment's partial alone."""
    _, cal_k, cal_v, kc, ka, vc, va, q = _setup(2, [1, 1], 64, n_q_heads=hq, n_kv_heads=2)
    R = cal_k[0].record_bytes
    qt = stored_to_torch(q).cuda()
    qt[:, 1, 5] = float("nan")
    g = torch.Generator().manual_seed(1)
    seg = [torch.randn((2, 2, 8, 128), generator=g).cuda() for _ in range(2)]
    out = torch.full((2, hq, 128), 7.0, device="cuda")
    ws = torch.zeros(P.aatc_decode_workspace_bytes(2, hq, 2, 64), dtype=torch.uint8, device="cuda")
    zero = torch.zeros(2, dtype=torch.int32, device="cuda")
    P.aatc_decode_attention_segmented(
        device_params(cal_k), device_params(cal_v), 2, hq, 2, qt, *[t.cuda() for t in (kc, ka, vc, va)],
        zero, 64, R, R, 128 ** -0.5, *seg, torch.tensor([5, 0], dtype=torch.int32, device="cuda"), 8, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(np.isnan(got[0, 1])) and np.all(np.isfinite(np.delete(got[0], 1, axis=0)))
    assert np.all(got[1] == 0)
