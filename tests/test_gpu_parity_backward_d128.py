"""Backward of heads of width 128 at the edges of its tiles: 32 rows or keys a wave and tile, two tiles a step of the
key-stationary kernel (odd counts leave one pair of waves without), 128 rows a workgroup of the row-stationary one."""
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,Hq,Hkv,alias,ns,win,block", [
    (1, 1, 1, 1, False, 0, 1, None),
    (1, 31, 1, 1, False, 0, 7, None),          # one tile: the second pair has none
    (2, 32, 2, 2, True, 1, None, None),
    (1, 65, 1, 1, False, 3, 40, None),         # three row tiles, a key tile of one key
    (1, 33, 32, 2, False, 5, 9, None),         # 16 heads a group: a tile is two positions
    (1, 130, 96, 1, False, 33, 50, None),      # 96 heads: a tile is a third of a position
    (2, 97, 16, 2, True, 0, 33, None),         # 8 heads a group
    (1, 161, 6, 3, False, 63, 65, None),       # the sink ends inside a wave's keys
    (1, 300, 4, 1, False, 1, 2, 48),           # blocks that are no multiple of a tile
    (1, 500, 8, 8, False, 40, 1, None),        # waves whose keys no row of a tile sees
])
def test_backward_d128_edges(gpu_device, B, S, Hq, Hkv, alias, ns, win, block):
    g = torch.Generator(device=gpu_device).manual_seed(91)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, k = r(B, S, Hq, 128), r(B, S, Hkv, 128)
    v, dout, scale = k if alias else r(B, S, Hkv, 128), r(B, S, Hq, 128), 128 ** -0.5
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, 128, block)
    got = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block)
    H.compare_backward(q, k, v, out, lse, dout, got, ns, win, scale, f"d128 bwd S{S} Hq{Hq}/{Hkv} ns{ns} W{win} b{block}", block)


@pytest.mark.parametrize("alias", [False, True])
@pytest.mark.parametrize("scale", [1e-25, 2e-30, 1.2e-38, 1e-40])
def test_scales_so_small_that_lse_over_scale_is_no_number(gpu_device, scale, alias):
    """Every live key has the same weight; below about 1e-37, lse / scale exceeds fp32."""
    S, ns, win = 300, 0, None
    g = torch.Generator(device=gpu_device).manual_seed(93)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, k, dout = r(1, S, 4, 128), r(1, S, 2, 128), r(1, S, 4, 128)
    v = k if alias else r(1, S, 2, 128)
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, 128, None)
    got = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, None)
    H.compare_backward(q, k, v, out, lse, dout, got, ns, win, scale, f"d128 bwd scale {scale} alias {alias}", None)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_bad_gradient_row_reaches_only_what_it_may(gpu_device, bad):
    """dout of one row of one head is not finite: dQ of the other rows is untouched, dK and dV of the keys it cannot see."""
    S, ns, win, scale, row = 200, 4, 30, 128 ** -0.5, 120
    g = torch.Generator(device=gpu_device).manual_seed(92)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, k, v, dout = r(1, S, 2, 128), r(1, S, 2, 128), r(1, S, 2, 128), r(1, S, 2, 128)
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, 128, None)
    clean = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, None)
    dirty = dout.clone()
    dirty[0, row, 1, 5] = bad
    got = H.run_backward(q, k, v, out, lse, dirty, ns, win, scale, None)
    ok_rows = torch.ones(S, 2, dtype=torch.bool, device=gpu_device)
    ok_rows[row, 1] = False
    assert torch.equal(got[0][0][ok_rows], clean[0][0][ok_rows])
    # (a key sees the row's zero weight through the whole tile of 32 rows: row 96 .. 127)
    ok_keys = torch.ones(S, 2, dtype=torch.bool, device=gpu_device)
    ok_keys[:128, 1] = False
    for a, b in zip(got[1:], clean[1:]):
        assert torch.equal(a[0][ok_keys], b[0][ok_keys])
