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
