"""Decode over tokens far outside the calibration's distribution: isotropic among strongly
anisotropic ones, so that a token's scale times the head's largest query weight is up to 600 (log2
domain) while its score is about 10.

The matrix-core scores take the query weights in fixed point, 27 bits or more below the head's
largest: each of up to 1000 set bits errs by at most 2^(3 - 31) of that largest weight, 4.6 / 8 and
1 / sqrt(3) of it at random, so a score by 600 x 2^-28 x 0.33 x sqrt(500) = 1.7e-5 (rms over the
wider records) and a weight by 0.7 of that.  An output averages the errors of its tokens: 1.2e-5
relative L2 per head.  (With 23 bits: 2.0e-5 to 6.6e-5.)"""
import numpy as np
import pytest
import torch

import paper_2608_14191_amd as P
from kvsynth import workload
from oracle import aatc as ora

from helpers import alpha_cache, device_params, record_cache, rel_l2, stored_to_torch, tile_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,bits,b_max", [(12, 2.75, 8), (16, 4.0, 8), (4, 5.0, 8), (7, 6.0, 12),
                                          (4, 7.0, 16), (12, 8.0, 16)])
def test_outlier_tokens(G, bits, b_max):
    print(f"[outliers] {G} {bits}", flush=True)
    H, lens, cap = 2, [3001, 515], 3008
    B, HQ = len(lens), H * G
    w = workload(2, n_tokens=max(lens), batch=B, n_kv_heads=H, n_q_heads=HQ)
    cal = {t: [ora.calibrate(w.calib(h, t), bits, b_max=b_max) for h in range(H)] for t in "kv"}
    R = {t: cal[t][0].record_bytes for t in "kv"}
    params = {t: device_params(cal[t]) for t in "kv"}
    codes = {"k": record_cache(H, cap, R["k"], batch=B), "v": tile_cache(H, cap, R["v"], batch=B)}
    alpha = {t: alpha_cache(H, cap, batch=B) for t in "kv"}
    for b in range(B):
        g = torch.Generator().manual_seed(b)
        for t, layout in (("k", P.LAYOUT_RECORDS), ("v", P.LAYOUT_TILES)):
            x = stored_to_torch(np.stack([w.cache(b, h, t) for h in range(H)], axis=1)).float()
            x[::16] = torch.randn(x[::16].shape, generator=g)
            P.aatc_encode(params[t], H, x.cuda(), lens[b], H * 128, layout, codes[t][b], alpha[t][b], cap, 0)
    q = np.stack([w.as_f32(w.queries(b)) for b in range(B)])
    out = torch.full((B, HQ, 128), float("nan"), device="cuda")
    ws = torch.zeros(P.aatc_decode_workspace_bytes(B, HQ, H, cap), dtype=torch.uint8, device="cuda")
    P.aatc_decode_attention(params["k"], params["v"], B, HQ, H, torch.from_numpy(q).float().cuda(),
                            codes["k"], alpha["k"], codes["v"], alpha["v"],
                            torch.tensor(lens, dtype=torch.int32, device="cuda"), cap, R["k"], R["v"],
                            128 ** -0.5, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    for b, n in enumerate(lens):
        for h in range(H):
            a = {t: alpha[t][b, h, :n].cpu().numpy().view(np.float16) for t in "kv"}
            k = ora.decode_tokens(codes["k"][b, h, :n].cpu().numpy(), a["k"], cal["k"][h])
            rec = ora.tiles_to_records(codes["v"][b, h].cpu().numpy(), R["v"])[:n]
            v = ora.decode_tokens(rec, a["v"], cal["v"][h])
            ref = ora.softmax_attention(q[b, h * G:(h + 1) * G].astype(np.float64), k, v, 128 ** -0.5)
            for j in range(G):
                err = rel_l2(got[b, h * G + j], ref[j])
                assert err <= 1.2e-5, (b, h, j, err)
