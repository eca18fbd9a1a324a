"""A tile of 128 query rows with a result of magnitude 2 has none of its rows from weights that are rounded to bf16 once.

Measured by the share of results that are not the 64-bit result rounded to bf16. With weights good to 2^-17 the error
before that rounding is about 2^-17 of a result, against a spacing of 2^-7 to 2^-8: some 0.2 % are the neighbour.
With weights rounded once (rms 2^-9.3 each) it is a third of the spacing: some 25 % are. The bound is 2 %.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_23966_amd as loza
from paper_2512_23966_amd import binding as B_
from tests import helpers as H
from tests.test_gpu_parity_extend import _rand, _run

pytestmark = pytest.mark.gpu


def _neighbours(q, kc, vc, out, rows, first, pattern, scale):
    """Share of the results of `rows` [(b, r, h)] that are not the correctly rounded ones; position first[b] + r."""
    rb, rr, rh = (np.asarray(x, dtype=np.int64) for x in zip(*rows))
    tb, tr, th = (torch.as_tensor(x, device=q.device) for x in (rb, rr, rh))
    ref, _ = oracle.ssa_rows(q[tb, tr, th].contiguous().cpu(), kc.cpu(), ("alias", out.shape[3]) if vc is kc else vc.cpu(), rb, rh,
                             np.asarray(first, dtype=np.int64)[rb] + rr, Hq=q.shape[2], n_sink=pattern[0], window=pattern[1], scale=scale)
    share = float((out[tb, tr, th].cpu() != torch.from_numpy(ref).to(torch.bfloat16)).double().mean())
    print(f"[neighbours] {share:.4f} of {len(rows)} rows", flush=True)
    return share


def test_wide_prefill_tile_with_a_large_result(gpu_device):
    S, pattern, scale = 700, (16, 500), 192 ** -0.5
    q, k = _rand((1, S, 64, 576), 71, torch.bfloat16, gpu_device), _rand((1, S, 1, 576), 72, torch.bfloat16, gpu_device)
    q[0, 600, 5] = 2 * k[0, 590, 0]                  # its weight sits on that key
    out, _ = H.run_prefill(q, k, k, *pattern, scale, d_v=512)
    assert out[0, 600, 5].abs().max() >= 2
    share = _neighbours(q, k, k, out, [(0, r, h) for r in (600, 601) for h in range(64)], [0], pattern, scale)
    assert share < 0.02


# the tile kernel; workgroups that share the keys of a tile (scratch memory), or one of them
@pytest.mark.parametrize("scratch", [False, True])
@pytest.mark.parametrize("d", [576, 128])
def test_extend_tile_with_a_large_result(gpu_device, d, scratch):
    B, Hq, Hkv, S_max, q_len, tile = (4, 64, 1, 6144, 33, 2) if d == 576 else (4, 32, 8, 2304, 70, 32)   # positions a tile
    d_v, pattern, scale = 512 if d == 576 else 128, (16, 5000 if d == 576 else 2000), (192 if d == 576 else 128) ** -0.5
    lens = [S_max, S_max - 7, S_max - 500, S_max - 1001]
    assert loza.loza_ssa_extend_workspace_bytes(B, Hq, Hkv, S_max, q_len, d, d_v, *pattern) > 0
    q, kc = _rand((B, q_len, Hq, d), 73, torch.bfloat16, gpu_device), _rand((B, S_max, Hkv, d), 74, torch.bfloat16, gpu_device)
    vc = kc if d == 576 else _rand((B, S_max, Hkv, d), 75, torch.bfloat16, gpu_device)
    r, h, G = 3, 5, Hq // Hkv
    q[0, r, h] = 2 * kc[0, S_max - 100, h // G]
    seqlens = torch.tensor(lens, dtype=torch.int32, device=gpu_device)
    if scratch:
        out, _ = _run(q, kc, vc, seqlens, pattern, scale, d_v)
    else:
        out, lse = torch.empty(B, q_len, Hq, d_v, dtype=torch.bfloat16, device=gpu_device), torch.empty(B, Hq, q_len, device=gpu_device)
        assert B_.lib().loza_ssa_extend(q.data_ptr(), kc.data_ptr(), vc.data_ptr(), seqlens.data_ptr(), out.data_ptr(), lse.data_ptr(), B, Hq, Hkv,
                                        S_max, q_len, d, d_v, *pattern, scale, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
    assert out[0, r, h].abs().max() >= 2
    r0 = r // tile * tile
    rows = [(0, x, y) for x in range(r0, r0 + tile) for y in range(h // G * G, h // G * G + G)]
    share = _neighbours(q, kc, vc, out, rows, [L - q_len for L in lens], pattern, scale)
    assert share < 0.02
