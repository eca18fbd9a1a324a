"""Backward where the key-stationary kernel cuts key tiles into chunks of rows for balance: few key tiles, all of
them cut (sink tiles in chunks or whole, ragged ends, separate and shared values, both patterns), and whole tiles
with a remainder beyond 256 in chunks, in one launch."""
import pytest
import torch

import paper_2512_23966_amd as loza
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _case(device, B, S, Hq, Hkv, d_qk, d_v, alias, seed=30):
    g = torch.Generator(device=device).manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device=device).to(torch.bfloat16)
    q, k = r(B, S, Hq, d_qk), r(B, S, Hkv, d_qk)
    return q, k, (k if alias else r(B, S, Hkv, d_v)), r(B, S, Hq, d_v)


@pytest.mark.parametrize("B,S,Hq,Hkv,d,alias,ns,win,block", [
    (1, 413, 32, 1, 128, False, 0, 150, None),    # no sink tile; the last key tile is ragged
    (1, 413, 32, 1, 128, False, 70, 100, None),   # sink tiles in chunks of their own, cut finer too
    (1, 413, 32, 1, 128, True, 70, None, None),   # every key live: one chunk per sink tile at the outset
    (2, 200, 64, 1, 576, True, 20, 90, None),     # (of the kernels that keep no weights in memory)
    (1, 333, 64, 1, 576, True, 1, 2, 64),         # block-granular
    (1, 1100, 4, 1, 128, False, 16, 600, None),   # nothing to cut: a chunk would be fewer than 32 row tiles
])
def test_backward_with_split_key_tiles(gpu_device, B, S, Hq, Hkv, d, alias, ns, win, block):
    d_v = 512 if d == 576 else 128
    q, k, v, dout = _case(gpu_device, B, S, Hq, Hkv, d, d_v, alias)
    scale, least = d ** -0.5, d == 576
    if S < 1000:
        assert loza.loza_ssa_backward_split(B, Hq, Hkv, S, d, d_v, ns, win, block or 1, alias)[0] >= 1
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, d_v, block)
    got = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block, least)
    H.compare_backward(q, k, v, out, lse, dout, got, ns, win, scale, f"split bwd S{S} Hq{Hq} d{d} ns{ns} W{win} b{block}", block)
    again = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block, least)
    assert all(a is b or torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(got, again))


# 256 whole items and a remainder in chunks: whole tiles numbered behind the cut ones, partial sums of sink tiles
# and of cut tiles side by side
@pytest.mark.parametrize("B,S,Hq,Hkv,alias,ns,win,block", [
    (2, 519, 64, 16, False, 20, 500, None),
    (4, 519, 32, 8, True, 0, 500, None),
    (2, 556, 64, 16, False, 2, 3, 128),
    (1, 1111, 64, 16, False, 20, 500, None),      # the sink tile in two chunks of its own
])
def test_backward_with_whole_and_split_key_tiles(gpu_device, B, S, Hq, Hkv, alias, ns, win, block):
    tiles, chunks, whole = loza.loza_ssa_backward_split(B, Hq, Hkv, S, 128, 128, ns, win, block or 1, alias)
    assert tiles >= 1 and chunks >= 2 and whole >= 256
    q, k, v, dout = _case(gpu_device, B, S, Hq, Hkv, 128, 128, alias, seed=31)
    scale = 128 ** -0.5
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, 128, block)
    got = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block)
    H.compare_backward(q, k, v, out, lse, dout, got, ns, win, scale, f"mixed bwd S{S} Hq{Hq} ns{ns} W{win} b{block}", block)
