"""Backward where the key-stationary kernel cuts key tiles into chunks of rows for balance (few key tiles, or
a remainder beyond full rounds of 256): sink tiles in chunks or whole, chunks that end up empty, ragged ends,
separate and shared values, both patterns."""
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
    (2, 200, 64, 1, 576, True, 20, 90, None),
    (1, 333, 64, 1, 576, True, 1, 2, 64),         # block-granular
    (1, 1100, 4, 1, 128, False, 16, 600, None),   # a chunk is 32 row tiles at least
])
def test_backward_with_split_key_tiles(gpu_device, B, S, Hq, Hkv, d, alias, ns, win, block):
    d_v = 512 if d == 576 else 128
    q, k, v, dout = _case(gpu_device, B, S, Hq, Hkv, d, d_v, alias)
    scale = d ** -0.5
    out, lse = H.oracle_forward_all(q, k, v, ns, win, scale, d_v, block)
    got = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block)
    H.compare_backward(q, k, v, out, lse, dout, got, ns, win, scale, f"split bwd S{S} Hq{Hq} d{d} ns{ns} W{win} b{block}", block)
    again = H.run_backward(q, k, v, out, lse, dout, ns, win, scale, block)
    assert all(a is b or torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(got, again))
