"""The full-precision segment's partial at the edges of its tiling: 64-token passes, the
largest segment, query groups of 1, 7 and 16, both input types, bases that are not 16-byte
aligned.  With no compressed tokens the output is the softmax over the segment alone, so the
reference is that attention in fp64.

Bound: scores of magnitude up to about 40 in fp32 are off by at most 40 2^-21 = 2e-5 absolute
(128-term dot products), hence the weights and the output by 4e-5 relative; 1e-4 with the sums.
"""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora

from helpers import alpha_cache, device_params, record_cache, rel_l2, stored_to_torch, tile_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("G", [1, 7, 16])
def test_segment_alone(G, dtype, off):
    counts, H, cap, seg_cap = [0, 1, 63, 64, 65, 200, 255, 256], 2, 64, 256
    B, HQ = len(counts), 2 * G
    w = workload(2, n_tokens=64, batch=B, n_kv_heads=H, n_q_heads=HQ)
    cal = [ora.calibrate(w.calib(h, "k"), 2.75) for h in range(H)]
    R = cal[0].record_bytes
    p = device_params(cal)
    kc, vc = record_cache(H, cap, R, batch=B), tile_cache(H, cap, R, batch=B)
    ka, va = alpha_cache(H, cap, batch=B), alpha_cache(H, cap, batch=B)
    g = torch.Generator().manual_seed(7 * G + off)
    n = B * H * seg_cap * 128

    def segment(scale):
        buf = torch.zeros(n + off, dtype=dtype)
        buf[off:] = (scale * torch.randn(n, generator=g)).to(dtype)
        return buf.cuda()[off:].view(B, H, seg_cap, 128)

    sk, sv = segment(2.0), segment(1.0)
    q = torch.randn((B, HQ, 128), generator=g).to(torch.bfloat16)
    zero = torch.zeros(B, dtype=torch.int32, device="cuda")
    st = torch.tensor(counts, dtype=torch.int32, device="cuda")
    out = torch.full((B, HQ, 128), float("nan"), device="cuda")
    ws = torch.zeros(P.aatc_decode_workspace_bytes(B, HQ, H, cap), dtype=torch.uint8, device="cuda")
    P.aatc_decode_attention_segmented(p, p, B, HQ, H, q.cuda(), kc, ka, vc, va, zero, cap, R, R,
                                      1 / np.sqrt(128), sk, sv, st, seg_cap, out, ws)
    torch.cuda.synchronize()
    got, k64, v64 = out.cpu().numpy(), sk.cpu().double().numpy(), sv.cpu().double().numpy()
    q64 = q.double().numpy()
    for b, m in enumerate(counts):
        for j in range(HQ):
            if m == 0:
                assert np.all(got[b, j] == 0)
                continue
            z = k64[b, j // G, :m] @ q64[b, j] / np.sqrt(128)
            e = np.exp(z - z.max())
            ref = e @ v64[b, j // G, :m] / e.sum()
            assert rel_l2(got[b, j], ref) <= 1e-4, (m, j)
