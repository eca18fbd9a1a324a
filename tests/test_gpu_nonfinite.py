"""Values that are not finite reach the queries that see them, as the plain sum of weight times value has it, and no
others. (The entry points ask for finite inputs; this is how far one that is not spreads.)"""
import numpy as np
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu


def _reference(q, k, v, pos, live, scale):
    """fp64 result of one query [d] over its live keys; 0 weights are dead keys and take no part."""
    s = (k[live].double() @ q.double()) * scale
    return torch.softmax(s, 0) @ v[live].double()


def _same_kind(got, ref, tol):
    got, ref = got.double().cpu(), ref.cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref))
    f = torch.isfinite(ref)
    assert float((got[f] - ref[f]).abs().max()) <= tol


@pytest.mark.parametrize("splits", [None, "1", "5"])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (6, 6), (32, 1)])
@pytest.mark.parametrize("L,ns,win", [(40, 3, 9), (300, 5, 200)])
def test_decode_values(gpu_device, monkeypatch, splits, Hq, Hkv, L, ns, win):
    if splits:
        monkeypatch.setenv("LOZA_DECODE_SPLITS", splits)
    B, d, scale = 3, 128, 128 ** -0.5
    g = torch.Generator(device=gpu_device).manual_seed(5)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, kc, vc = r(B, Hq, d), r(B, L, Hkv, d), r(B, L, Hkv, d)
    inf, nan = float("inf"), float("nan")
    vc[0, L - 2, :, 3], vc[0, 1, :, 70], vc[0, L - 4, :, 71] = inf, -inf, nan     # live keys
    vc[0, L - 3, :, 72], vc[0, L - 5, :, 72] = inf, -inf
    vc[1, ns:L - win] = nan                                                          # dead ones, some in a live tile
    lens = torch.full((B,), L, dtype=torch.int32, device=gpu_device)
    out, lse = H.run_decode(q, kc, vc, lens, ns, win, scale)
    live = torch.tensor(list(range(ns)) + list(range(L - win, L)), device=gpu_device)
    ref = torch.stack([torch.stack([_reference(q[b, h], kc[b, :, h * Hkv // Hq], vc[b, :, h * Hkv // Hq], L - 1, live, scale)
                                    for h in range(Hq)]) for b in range(B)])
    assert int(torch.isinf(ref).sum()) == 2 * Hq and int(torch.isnan(ref).sum()) == 2 * Hq
    _same_kind(out, ref, 1e-2)
    assert bool(torch.isfinite(lse).all())


@pytest.mark.parametrize("d_qk,d_v", [(64, 64), (100, 66), (200, 130), (256, 255)])
@pytest.mark.parametrize("S,Hq,Hkv,ns,win", [(75, 2, 1, 5, 20), (140, 3, 3, 0, 33)])
def test_f32_values(gpu_device, d_qk, d_v, S, Hq, Hkv, ns, win):
    g = torch.Generator(device=gpu_device).manual_seed(6)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device)
    q, k, v, scale = r(1, S, Hq, d_qk), r(1, S, Hkv, d_qk), r(1, S, Hkv, d_v), d_qk ** -0.5
    inf, nan = float("inf"), float("nan")
    v[0, 41, :, 3], v[0, 50, :, 5], v[0, 50, :, 3], v[0, 2, :, 60] = inf, nan, -inf, -inf
    k[0, 44] = nan
    q[0, 30, 0] = nan
    out, lse = H.run_prefill(q, k, v, ns, win, scale)
    kc, vc, lens = k, v, torch.tensor([S], dtype=torch.int32, device=gpu_device)
    out_d, lse_d = H.run_decode_f32(q[:, S - 1].contiguous(), kc, vc, lens, ns, win, scale)
    dev = gpu_device
    ref = torch.empty(1, S, Hq, d_v, dtype=torch.float64, device=dev)
    for i in range(S):
        live = torch.tensor(sorted(set(range(min(ns, i + 1))) | set(range(max(0, i - win + 1), i + 1))), device=dev)
        for h in range(Hq):
            ref[0, i, h] = _reference(q[0, i, h], k[0, :, h * Hkv // Hq], v[0, :, h * Hkv // Hq], i, live, scale)
    assert 0 < int(torch.isnan(ref).sum()) < ref.numel() // 2 and int(torch.isinf(ref).sum()) > 0
    _same_kind(out, ref, 1e-5)
    _same_kind(out_d, ref[:, S - 1], 1e-5)
    assert torch.equal(torch.isnan(lse[0].T), torch.isnan(ref[0]).all(-1))


def test_f32_scores_that_are_all_minus_infinity(gpu_device):
    """Finite inputs whose products overflow: -inf for every live key has no softmax (NaN, not a silent 0)."""
    q, k = torch.full((1, 20, 1, 8), 3e20, device=gpu_device), torch.full((1, 20, 1, 8), -3e20, device=gpu_device)
    v = torch.ones(1, 20, 1, 8, device=gpu_device)
    out, lse = H.run_prefill(q, k, v, 1, 4, 1.0)
    assert bool(torch.isnan(out).all()) and bool(torch.isnan(lse).all())
