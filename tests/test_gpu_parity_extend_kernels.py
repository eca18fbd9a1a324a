"""Extends and prompts of few rows by the kernels that took them over: at the wide shape, tiles of 128 rows whose keys are
split, for calls that the few-rows kernel serves where there is no scratch memory; at width 128, the few-rows
kernel with 32 rows a workgroup, for more groups of 16 than compute units."""
import numpy as np
import pytest
import torch

import paper_2512_23966_amd as loza
from paper_2512_23966_amd.binding import KERNEL_ROWS
from tests import helpers as H
from tests.test_gpu_parity_extend import _rand
from tests.test_gpu_parity_extend_split import _check, _plan

pytestmark = pytest.mark.gpu


def _extend(device, B, Hq, Hkv, d, S_max, q_len, lens, ns, win, block, label, step):
    q, kc = _rand((B, q_len, Hq, d), 81, torch.bfloat16, device), _rand((B, S_max, Hkv, d), 82, torch.bfloat16, device)
    vc = kc if d == 576 else _rand((B, S_max, Hkv, d), 83, torch.bfloat16, device)
    for b, L in enumerate(lens):
        kc[b, L:] = float("nan")
        vc[b, L:] = float("nan")
    seqlens, scale, d_v = torch.tensor(lens, dtype=torch.int32, device=device), (192 if d == 576 else 128) ** -0.5, 512 if d == 576 else 128
    out = torch.full((B, q_len, Hq, d_v), float("nan"), dtype=torch.bfloat16, device=device)
    lse = torch.full((B, Hq, q_len), float("nan"), dtype=torch.float32, device=device)
    if block:
        loza.loza_ssa_extend_blocks(q, kc, vc, seqlens, out, lse, ns, win, block, scale)
    else:
        loza.loza_ssa_extend(q, kc, vc, seqlens, out, lse, ns, win, scale)
    _check(q, kc, vc, lens, out, lse, (ns, win), scale, label, block, step)


@pytest.mark.parametrize("B,S_max,q_len,lens,ns,win,block,step", [
    (2, 6000, 16, [6000, 5555], 128, 5000, None, 3),        # 128 groups of 16 rows
    (5, 2700, 15, [2700, 2600, 700, 9, 0], 0, 2500, None, 5),   # 300 groups; queries before the start; an empty cache
    (4, 2600, 17, [2600, 2599, 140, 18], 3, 16, 128, 5),    # blocks; half a tile at the end
])
def test_tiles_of_few_rows(gpu_device, B, S_max, q_len, lens, ns, win, block, step):
    n, groups = _plan(B, 64, 1, S_max, q_len, 576, ns, win, block or 1), q_len * 4 * B
    assert groups <= 512 and n > 1 and n * groups > 256     # more parts than the few-rows kernel would be cut into
    _extend(gpu_device, B, 64, 1, 576, S_max, q_len, lens, ns, win, block, f"tiles of few rows q{q_len} n{n}", step)


@pytest.mark.parametrize("B,Hq,Hkv,S_max,q_len,lens,ns,win,block", [
    (1, 32, 8, 700, 130, [700], 20, 90, None),              # 33 groups a key head: the last pair is half a group
    (3, 12, 4, 600, 181, [600, 200, 3], 0, 130, None),      # 3 heads a group; queries before the start
    (1, 64, 32, 500, 121, [500], 1, 2, 48),                 # 2 heads a group, blocks; two rows in the last group
])
def test_pairs_of_row_groups(gpu_device, B, Hq, Hkv, S_max, q_len, lens, ns, win, block):
    groups = (q_len * (Hq // Hkv) + 15) // 16 * Hkv * B
    assert 256 < groups <= 512 and (q_len * (Hq // Hkv) + 31) // 32 * Hkv * B <= 256 and _plan(B, Hq, Hkv, S_max, q_len, 128, ns, win, block or 1) == 1
    _extend(gpu_device, B, Hq, Hkv, 128, S_max, q_len, lens, ns, win, block, f"pairs {Hq}/{Hkv} q{q_len}", 3)


@pytest.mark.parametrize("S,Hq,Hkv,alias", [(130, 32, 8, False), (1100, 4, 1, True), (81, 64, 64, False)])
def test_prompts_of_paired_row_groups(gpu_device, S, Hq, Hkv, alias):
    q, k = _rand((1, S, Hq, 128), 84, torch.bfloat16, gpu_device), _rand((1, S, Hkv, 128), 85, torch.bfloat16, gpu_device)
    v = k if alias else _rand((1, S, Hkv, 128), 86, torch.bfloat16, gpu_device)
    assert loza.loza_ssa_forward_kernel(1, Hq, Hkv, S, S, 128, 16, 50, 1) == KERNEL_ROWS and (S * (Hq // Hkv) + 15) // 16 * Hkv > 256
    out, lse = H.run_prefill(q, k, v, 16, 50, 128 ** -0.5)
    rb, rh, ri = H.all_rows(1, Hq, S)
    H.compare_prefill(q, k, v, out, lse, rb, rh, ri, 16, 50, 128 ** -0.5, f"paired groups S{S} {Hq}/{Hkv}")
