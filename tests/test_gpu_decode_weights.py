"""Decode weights are not rounded: queries whose result cancels to far below their values show every bit a weight
loses. A query with few live keys, and one whose weight sits on few keys with a result of magnitude 2 and more in
some column, are such."""
import numpy as np
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [None, "1", "5"])
@pytest.mark.parametrize("d_qk,d_v,alias,heads", [(576, 512, True, 1), (128, 128, False, 6)])
@pytest.mark.parametrize("L,ns,win", [(9, 2, 4), (100, 30, 40), (700, 40, 600)])
def test_decode_results_that_cancel(gpu_device, monkeypatch, splits, d_qk, d_v, alias, heads, L, ns, win):
    if splits:
        monkeypatch.setenv("LOZA_DECODE_SPLITS", splits)
    B, r = 12, np.random.default_rng(L + d_qk)
    q = torch.zeros(B, heads, d_qk, dtype=torch.bfloat16)
    q[..., d_qk - 1] = 1.0                                  # the score of a key is its last feature
    kc = torch.zeros(B, L, heads, d_qk, dtype=torch.bfloat16)
    vc = kc if alias else torch.zeros(B, L, heads, d_v, dtype=torch.bfloat16)
    vc[..., :d_v] = torch.from_numpy(r.choice([-1, 1], (B, L, heads, d_v)) * r.uniform(64, 256, (B, L, heads, d_v)))
    scale = float(np.float32(np.log(2.0)))                  # scores are powers of 2, exactly
    live = np.r_[0:ns, L - win:L]
    s = r.integers(-16, 0, (B, L, heads)) / 8.0
    hot = live[-7:]                                         # nearly all the weight where keys are many
    s[:, hot] += 8.0 if L > 128 else 0.0
    kc[..., d_qk - 1] = torch.from_numpy(s)
    p = np.exp2(s[:, live] * np.log2(np.e) * scale)
    p /= p.sum(1, keepdims=True)
    # the last four keys cancel what the others add up to, each but for the rounding of its values to bf16
    for x in range(4):
        j = len(live) - 4 + x
        vals = vc[:, live][..., :d_v].double().numpy()
        rest = (p[..., None] * vals).sum(1) - p[:, j, :, None] * vals[:, j]
        rest[..., 0] = 0.0                                  # (a large result in column 0)
        vc[:, live[j], :, :d_v] = torch.from_numpy(-rest / p[:, j, :, None]).to(torch.bfloat16)
    q, kc = q.to(gpu_device), kc.to(gpu_device)
    vc = kc if alias else vc.to(gpu_device)
    lens = torch.full((B,), L, dtype=torch.int32, device=gpu_device)
    out, lse = H.run_decode(q, kc, vc, lens, ns, win, scale, d_v=d_v)
    rb, rh = np.repeat(np.arange(B), heads), np.tile(np.arange(heads), B)
    ref, ref_lse = H.oracle_decode(q, kc, vc, lens, rb, rh, ns, win, scale, d_v)
    got = out[torch.as_tensor(rb, device=gpu_device), torch.as_tensor(rh, device=gpu_device)].double().cpu().numpy()
    mass = (p[..., None] * np.abs(vc[:, torch.as_tensor(live, device=gpu_device)][..., :d_v].double().cpu().numpy())).sum(1).reshape(ref.shape)
    err = np.abs(got - ref)
    # the result is rounded to bf16 (half an ulp); before that every weight carries the exponential's rounding (one
    # ulp, 2^-23) and the fp32 sums a few of 2^-24, against the weighted sum of the values' magnitudes. Two bf16
    # terms (2^-18 a weight, a handful of weights) leave 2^-20 and more.
    half_ulp = np.exp2(np.floor(np.log2(np.abs(ref) + 1e-30)) - 8)
    units = (err - half_ulp) / mass * 2.0 ** 24
    print(f"[parity] cancel L{L} d{d_qk} splits{splits}: worst {units.max():.2f} units of 2^-24 (bound 8)", flush=True)
    assert units.max() <= 8.0
    assert np.abs(ref[:, 0]).max() > 2.0
    assert np.abs(lse[torch.as_tensor(rb, device=gpu_device), torch.as_tensor(rh, device=gpu_device)].double().cpu().numpy() - ref_lse).max() <= 2e-5
