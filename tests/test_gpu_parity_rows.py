"""The few-rows kernel (decode, short extends and prompts) where it can go wrong: lengths around its 16-key
tiles, sink and window edges inside a tile, fewer tiles than waves, groups of 16 rows that straddle positions
or are partly empty, row counts on both sides of the line to the tile kernel, one split and many."""
import numpy as np
import pytest
import torch

import paper_2512_23966_amd as loza
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _rand(shape, seed, device):
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.randn(shape, generator=g, device=device, dtype=torch.float32).to(torch.bfloat16)


LENS = [1, 15, 16, 17, 31, 33, 64, 65, 0, 127, 128, 129, 300, 511]


@pytest.mark.parametrize("splits", [None, "1", "7"])
@pytest.mark.parametrize("Hq,Hkv,d_qk,d_v,alias", [(64, 1, 576, 512, True), (20, 1, 576, 512, True), (8, 2, 128, 128, False),
                                                   (64, 1, 128, 128, True), (6, 6, 128, 128, False)])
@pytest.mark.parametrize("ns,win,block", [(5, 40, None), (128, 300, None), (0, 1, None), (1, 2, 48), (16, None, None)])
def test_decode_lengths_around_the_tile(gpu_device, monkeypatch, splits, Hq, Hkv, d_qk, d_v, alias, ns, win, block):
    if splits:
        monkeypatch.setenv("LOZA_DECODE_SPLITS", splits)
    B, S_max, scale = len(LENS), 511, d_qk ** -0.5
    q, kc = _rand((B, Hq, d_qk), 1, gpu_device), _rand((B, S_max, Hkv, d_qk), 2, gpu_device)
    vc = kc if alias else _rand((B, S_max, Hkv, d_v), 3, gpu_device)
    for b, L in enumerate(LENS):
        kc[b, L:] = float("nan")   # rows at or beyond the length must never be read
        vc[b, L:] = float("nan")
    lens = torch.tensor(LENS, dtype=torch.int32, device=gpu_device)
    out, lse = H.run_decode(q, kc, vc, lens, ns, win, scale, d_v=d_v, block=block)
    z = LENS.index(0)
    assert bool((out[z] == 0).all()) and bool(torch.isneginf(lse[z]).all())
    live = [b for b in range(B) if LENS[b]]
    rb, rh = np.repeat(np.asarray(live, dtype=np.int64), Hq), np.tile(np.arange(Hq, dtype=np.int64), len(live))
    H.compare_decode(q, kc, vc, lens, out, lse, rb, rh, ns, win, scale, f"rows decode {Hq}/{Hkv} d{d_qk} {ns},{win},{block}", block)


# groups of 16 rows: 512 take the row kernel, 513 and more the tile kernel
@pytest.mark.parametrize("B,q_len,Hq,Hkv,d,alias", [(1, 128, 64, 1, 576, True), (1, 129, 64, 1, 576, True), (3, 7, 12, 1, 576, True),
                                                    (2, 5, 3, 1, 128, False), (1, 64, 32, 8, 128, False)])
def test_extend_row_groups(gpu_device, B, q_len, Hq, Hkv, d, alias):
    S_max, ns, win, scale = 400, 20, 90, d ** -0.5
    d_v = 512 if d == 576 else 128
    lens_h = [S_max - 37 * b for b in range(B)]
    lens_h[-1] = max(1, min(lens_h[-1], q_len - 1))   # some queries of the last sequence lie before its start
    q, kc = _rand((B, q_len, Hq, d), 4, gpu_device), _rand((B, S_max, Hkv, d), 5, gpu_device)
    vc = kc if alias else _rand((B, S_max, Hkv, d_v), 6, gpu_device)
    lens = torch.tensor(lens_h, dtype=torch.int32, device=gpu_device)
    out = torch.full((B, q_len, Hq, d_v), float("nan"), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.full((B, Hq, q_len), float("nan"), dtype=torch.float32, device=gpu_device)
    loza.loza_ssa_extend(q, kc, vc, lens, out, lse, ns, win, scale)
    torch.cuda.synchronize()
    for b, L in enumerate(lens_h):
        for r in range(q_len):
            i = L - q_len + r
            if i < 0:
                assert bool((out[b, r] == 0).all()) and bool(torch.isneginf(lse[b, :, r]).all())
        first = max(0, q_len - L)
        rows = np.asarray([(h, r) for h in range(Hq) for r in range(first, q_len)], dtype=np.int64)
        rh, rr = rows[:, 0].copy(), rows[:, 1].copy()
        zero = np.zeros_like(rh)
        qf = torch.zeros(1, L, Hq, d, dtype=torch.bfloat16, device=gpu_device)
        of = torch.zeros(1, L, Hq, d_v, dtype=torch.bfloat16, device=gpu_device)
        lf = torch.zeros(1, Hq, L, dtype=torch.float32, device=gpu_device)
        n = q_len - first
        qf[0, L - n:], of[0, L - n:], lf[0, :, L - n:] = q[b, first:], out[b, first:], lse[b, :, first:]
        kb = kc[b:b + 1, :L].contiguous()
        vb = kb if alias else vc[b:b + 1, :L].contiguous()
        H.compare_prefill(qf, kb, vb, of, lf, zero, rh, rr + L - q_len, ns, win, scale, f"rows extend q{q_len} {Hq}/{Hkv} d{d} L{L}")


# fp32 twin: its blocks of 64 features and columns, widths that are no multiple of 4 (guarded scalar loads)
@pytest.mark.parametrize("d_qk,d_v", [(1, 1), (3, 66), (63, 64), (64, 65), (128, 4), (129, 130), (192, 192), (193, 7), (256, 255), (256, 256)])
@pytest.mark.parametrize("S,Hq,Hkv,ns,win", [(17, 1, 1, 2, 3), (50, 6, 2, 20, 16)])
def test_prefill_f32_widths(gpu_device, d_qk, d_v, S, Hq, Hkv, ns, win):
    g = torch.Generator(device=gpu_device).manual_seed(7)
    q, k, v = (torch.randn(2, S, h, d, generator=g, device=gpu_device) for h, d in ((Hq, d_qk), (Hkv, d_qk), (Hkv, d_v)))
    scale = d_qk ** -0.5
    out, lse = H.run_prefill(q, k, v, ns, win, scale)
    rb, rh, ri = H.all_rows(2, Hq, S)
    H.compare_prefill(q, k, v, out, lse, rb, rh, ri, ns, win, scale, f"f32 widths {d_qk},{d_v} S{S}")


# Heads of width 128, more rows than that: tiles of 128 rows (the 256-row kernel's cases are in
# test_gpu_parity_kernels_by_size.py); ragged ends, sink and window edges inside a step of 32 keys, whole tiles of
# two-term weights, shared and separate values
@pytest.mark.parametrize("B,S,Hq,Hkv,alias,ns,win,block", [
    (2, 277, 160, 40, False, 37, 70, None),      # the last row tile is ragged
    (1, 530, 128, 64, True, 0, 200, None),
    (1, 600, 96, 96, False, 1, 3, 48),
    (3, 300, 64, 64, False, 128, None, None),    # a last tile of 44 rows
    (1, 300, 40, 40, False, 5, 33, None),
])
def test_d128_prefill_tiles(gpu_device, B, S, Hq, Hkv, alias, ns, win, block):
    q, k = _rand((B, S, Hq, 128), 11, gpu_device), _rand((B, S, Hkv, 128), 12, gpu_device)
    v = k if alias else _rand((B, S, Hkv, 128), 13, gpu_device)
    scale = 128 ** -0.5
    out, lse = H.run_prefill(q, k, v, ns, win, scale, d_v=128, block=block)
    rb, rh, ri = H.all_rows(B, Hq, S)
    keep = (rh % 7 == 0) | (rh == Hq - 1)
    H.compare_prefill(q, k, v, out, lse, rb[keep], rh[keep], ri[keep], ns, win, scale, f"d128 tiles S{S} {Hq}/{Hkv}", block)


def test_d128_extend_paged_of_32_rows(gpu_device):
    """Pages of 32 rows; peaked rows take the two-term pass."""
    B, q_len, H_, S_max, page, ns, win, scale = 2, 500, 48, 640, 32, 40, 150, 128 ** -0.5
    lens_h = [S_max - 3, 555]
    q, kc, vc = _rand((B, q_len, H_, 128), 14, gpu_device), _rand((B, S_max, H_, 128), 15, gpu_device), _rand((B, S_max, H_, 128), 16, gpu_device)
    q[:, 100::50] *= 6
    lens = torch.tensor(lens_h, dtype=torch.int32, device=gpu_device)
    perm = torch.randperm(B * S_max // page, generator=torch.Generator().manual_seed(5)).to(torch.int32).view(B, -1)
    pools = []
    for c in (kc, vc):
        pool = torch.empty(B * S_max // page, page, H_, 128, dtype=torch.bfloat16, device=gpu_device)
        pool[perm.flatten().long().to(gpu_device)] = c.view(-1, page, H_, 128)
        pools.append(pool)
    res = []
    for paged in (False, True):
        out = torch.full((B, q_len, H_, 128), float("nan"), dtype=torch.bfloat16, device=gpu_device)
        lse = torch.full((B, H_, q_len), float("nan"), dtype=torch.float32, device=gpu_device)
        if paged:
            loza.loza_ssa_extend_paged(q, pools[0], pools[1], perm.to(gpu_device), lens, out, lse, ns, win, scale)
        else:
            loza.loza_ssa_extend(q, kc, vc, lens, out, lse, ns, win, scale)
        torch.cuda.synchronize()
        res.append((out, lse))
    assert torch.equal(res[0][0].view(torch.int16), res[1][0].view(torch.int16)) and torch.equal(res[0][1], res[1][1])
    for b, L in enumerate(lens_h):
        qf = torch.zeros(1, L, H_, 128, dtype=torch.bfloat16, device=gpu_device)
        of, lf = torch.zeros_like(qf), torch.zeros(1, H_, L, dtype=torch.float32, device=gpu_device)
        qf[0, L - q_len:], of[0, L - q_len:], lf[0, :, L - q_len:] = q[b], res[0][0][b], res[0][1][b]
        rows = np.asarray([(h, i) for h in (0, 17, H_ - 1) for i in range(L - q_len, L)], dtype=np.int64)
        H.compare_prefill(qf, kc[b:b + 1, :L].contiguous(), vc[b:b + 1, :L].contiguous(), of, lf, np.zeros(len(rows), dtype=np.int64),
                          rows[:, 0].copy(), rows[:, 1].copy(), ns, win, scale, f"d128 extend L{L}")


def test_decode_tile_kernel_recomputes_large_results(gpu_device):
    """Many sequences on a long window of 64 heads take the tile kernel, whose weights are rounded once: queries
    whose weight sits on one key (results of magnitude 2 and more) and queries with few live keys are recomputed."""
    B, Hq, S_max, ns, win, scale = 40, 64, 8600, 128, 8192, 192 ** -0.5
    q, kc = _rand((B, Hq, 576), 21, gpu_device), _rand((B, S_max, 1, 576), 22, gpu_device)
    lens_h = [S_max - 11 * b for b in range(B)]
    lens_h[3], lens_h[7], lens_h[9] = 100, 1, 0
    # three heads follow one key each: score about 0.35 * 576 / sqrt(192) = 14.5, i.e. 99 % of the weight
    for b in (0, 5, 11):
        for h, j in ((0, 5), (33, lens_h[b] - 1), (63, lens_h[b] - 4000)):
            q[b, h] = 0.35 * kc[b, j, 0]
    lens = torch.tensor(lens_h, dtype=torch.int32, device=gpu_device)
    out, lse = H.run_decode(q, kc, kc, lens, ns, win, scale, d_v=512)
    rb = np.repeat(np.asarray([0, 3, 5, 7, 11], dtype=np.int64), Hq)
    rh = np.tile(np.arange(Hq, dtype=np.int64), 5)
    assert bool((out[0].abs() >= 2).any())
    ref_out, ref_lse = H.oracle_decode(q, kc, kc, lens, rb, rh, ns, win, scale, 512)
    idx = (torch.as_tensor(rb, device=gpu_device), torch.as_tensor(rh, device=gpu_device))
    err = np.abs(out[idx].double().cpu().numpy() - ref_out)
    assert (err <= H.out_tolerance(ref_out, torch.bfloat16)).all(), err.max()
    # a recomputed score is one fp32 sum of 576 terms, each rounding at most half an ulp of a partial sum below 16
    assert np.abs(lse[idx].double().cpu().numpy() - ref_lse).max() <= 576 * 2.0 ** -24 * 16
