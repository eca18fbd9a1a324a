"""Every form of the kernels that large calls take, at sizes the oracle can follow: the tile kernel's decode, the
256-row and the 128-row kernel of width 128. The small cases of the other files run the few-rows kernel; each case
here says on the host which kernel it runs."""
import numpy as np
import pytest
import torch

import paper_2512_23966_amd as loza
from paper_2512_23966_amd import KERNEL_D128, KERNEL_TILES
from tests import helpers as H
from tests.test_gpu_canary import Guarded, _all_written

pytestmark = pytest.mark.gpu


def _rand(shape, seed, device):
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.randn(shape, generator=g, device=device, dtype=torch.float32).to(torch.bfloat16)


# ---- decode, tile kernel: many sequences on key heads of more than 32 query heads -------------------------

@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,d,alias,S_max,ns,win,block,n_splits", [
    (260, 64, 1, 576, True, 1344, 128, 1024, None, 1),
    (128, 64, 1, 576, True, 1536, 1, 7, 128, 2),
    (128, 48, 1, 576, True, 2304, 16, 2048, None, 2),
    (40, 128, 2, 128, False, 8448, 128, 8192, None, 3),
    (64, 48, 1, 128, True, 8448, 0, 8192, None, 4),
    (260, 128, 1, 128, False, 2112, 1, 8, 256, 1),
])
def test_decode_tile_kernel(gpu_device, paged, B, Hq, Hkv, d, alias, S_max, ns, win, block, n_splits):
    assert loza.loza_ssa_decode_kernel(B, Hq, Hkv, S_max, d, ns, win, block or 1) == (KERNEL_TILES, n_splits)
    d_v, scale, page = 512 if d == 576 else 128, (192 if d == 576 else 128) ** -0.5, 64
    kc = _rand((B, S_max, Hkv, d), 1, gpu_device)
    vc = kc if alias else _rand((B, S_max, Hkv, d_v), 2, gpu_device)
    q = _rand((B, Hq, d), 3, gpu_device)
    lens_h = [S_max - 5 * b for b in range(B)]
    lens_h[B - 1] = S_max - 7
    lens_h[2], lens_h[3], lens_h[4], lens_h[5] = 0, 1, 100, 130     # empty; computed directly; just not
    # heads that follow one key, a long way back and the newest: results of magnitude 2 and more
    c = 0.4 if d == 576 else 1.6
    for b in (0, 6, B - 1):
        for h, j in ((0, lens_h[b] - 1), (Hq // 2, lens_h[b] - 300), (Hq - 1, lens_h[b] - 40)):
            q[b, h] = (c * kc[b, j, h * Hkv // Hq].float()).to(torch.bfloat16)
    for b in range(B):
        kc[b, lens_h[b]:] = float("nan")
        vc[b, lens_h[b]:] = float("nan")
    lens = torch.tensor(lens_h, dtype=torch.int32, device=gpu_device)
    if paged:
        per = S_max // page
        perm = torch.randperm(B * per, generator=torch.Generator().manual_seed(4)).to(torch.int32)
        k_pool = torch.empty(B * per, page, Hkv, d, dtype=torch.bfloat16, device=gpu_device)
        k_pool[perm.long().to(gpu_device)] = kc.view(-1, page, Hkv, d)
        v_pool = k_pool
        if not alias:
            v_pool = torch.empty(B * per, page, Hkv, d_v, dtype=torch.bfloat16, device=gpu_device)
            v_pool[perm.long().to(gpu_device)] = vc.view(-1, page, Hkv, d_v)
        from tests.test_gpu_parity_paged import _run_paged
        out, lse = _run_paged(q, k_pool, v_pool, perm.view(B, per).to(gpu_device), lens, ns, win, scale, d_v, block)
    else:
        out, lse = H.run_decode(q, kc, vc, lens, ns, win, scale, d_v=d_v, block=block)
    assert bool((out[2] == 0).all()) and bool(torch.isneginf(lse[2]).all())
    assert int((out[0].abs() >= 2).sum()) > 0, "the construction no longer makes large results"
    sel = np.asarray([0, 3, 4, 5, 6, 17, B - 1], dtype=np.int64)
    rb, rh = np.repeat(sel, Hq), np.tile(np.arange(Hq, dtype=np.int64), len(sel))
    ref, ref_lse = H.oracle_decode(q, kc, vc, lens, rb, rh, ns, win, scale, d_v, block)
    idx = (torch.as_tensor(rb, device=gpu_device), torch.as_tensor(rh, device=gpu_device))
    err = np.abs(out[idx].double().cpu().numpy() - ref)
    assert (err <= H.out_tolerance(ref, torch.bfloat16)).all(), float((err - H.out_tolerance(ref, torch.bfloat16)).max())
    # a score computed directly is one fp32 sum of d terms, each rounding at most half an ulp of a partial sum below 32
    assert np.abs(lse[idx].double().cpu().numpy() - ref_lse).max() <= d * 2.0 ** -24 * 32


# ---- width 128, many rows ------------------------------------------------------------------------------------

# (B, S, Hq, Hkv, alias, n_sink, window, block): one list per kernel
D128_CASES = [
    (1, 1000, 64, 64, False, 100, None, None),
    (2, 517, 192, 24, False, 37, 300, None),        # eight heads on a key head; ragged
    (1, 900, 128, 16, True, 0, 333, None),
    (1, 1023, 192, 24, False, 2, 5, 96),
    (1, 700, 256, 32, True, 1, 2, 128),
]
TILE_CASES = [
    (1, 300, 40, 40, False, 37, 70, None),
    (2, 257, 24, 24, True, 0, 200, None),
    (1, 530, 36, 12, False, 3, 4, 48),
    (1, 420, 64, 64, False, 16, 100, None),
    (1, 1000, 64, 8, False, 0, 60, None),            # few live keys: two-term weights throughout
]


def _kernel(c, queries=None):
    B, S, Hq, Hkv, _, ns, win, block = c
    return loza.loza_ssa_forward_kernel(B, Hq, Hkv, queries or S, S, 128, ns, win, block or 1)


def _inputs(c, device, hot=1.0):
    B, S, Hq, Hkv, alias = c[:5]
    q, k = _rand((B, S, Hq, 128), 5, device), _rand((B, S, Hkv, 128), 6, device)
    return (q.float() * hot).to(torch.bfloat16), k, (k if alias else _rand((B, S, Hkv, 128), 7, device))


def _rows(c):
    """All positions of a few heads."""
    B, S, Hq = c[:3]
    rb, rh, ri = H.all_rows(B, Hq, S)
    keep = np.isin(rh, [0, 1, Hq // 2 + 1, Hq - 1])
    return rb[keep], rh[keep], ri[keep]


@pytest.mark.parametrize("hot", [1.0, 3.0])          # (times 3: the softmax reference moves all the time, large results)
@pytest.mark.parametrize("kernel,c", [(KERNEL_D128, c) for c in D128_CASES] + [(KERNEL_TILES, c) for c in TILE_CASES])
def test_d128_prefill(gpu_device, kernel, c, hot):
    assert _kernel(c) == kernel
    q, k, v = _inputs(c, gpu_device, hot)
    ns, win, block = c[5:]
    scale = 128 ** -0.5
    out, lse = H.run_prefill(q, k, v, ns, win, scale, d_v=128, block=block)
    H.compare_prefill(q, k, v, out, lse, *_rows(c), ns, win, scale, f"d128 kernel {kernel} {c} hot{hot}", block)
    # a chunk that is the whole sequence: the extend form of the same kernel, same bits
    B, S = c[:2]
    o2, l2 = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    sl = torch.full((B,), S, dtype=torch.int32, device=gpu_device)
    if block is None:
        loza.loza_ssa_extend(q, k, v, sl, o2, l2, ns, win, scale)
    else:
        loza.loza_ssa_extend_blocks(q, k, v, sl, o2, l2, ns, win, block, scale)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse.view(torch.int32), l2.view(torch.int32))


@pytest.mark.parametrize("kernel,c,q_len", [
    (KERNEL_D128, (2, 1500, 192, 24, False, 40, 500, None), 260), (KERNEL_D128, (2, 1500, 192, 24, True, 1, 5, 96), 260),
    (KERNEL_TILES, (2, 700, 24, 24, True, 40, 150, None), 250), (KERNEL_TILES, (2, 700, 24, 24, False, 0, 3, 64), 250)])
def test_d128_extend(gpu_device, kernel, c, q_len):
    """Ragged caches, NaN beyond each length; one shorter than the chunk. Outputs between guard zones. The same rows
    in pages of 32 give the same bits."""
    B, S, Hq, Hkv, alias, ns, win, block = c
    assert _kernel(c, q_len) == kernel
    q, k, v = _inputs(c, gpu_device)
    q = q[:, :q_len].contiguous()
    lens = [S - 3, q_len - 40]
    for b, L in enumerate(lens):
        k[b, L:] = float("nan")
        v[b, L:] = float("nan")
    G = Guarded(gpu_device)
    out, lse = G.tensor((B, q_len, Hq, 128), torch.bfloat16), G.tensor((B, Hq, q_len), torch.float32)
    sl, scale = torch.tensor(lens, dtype=torch.int32, device=gpu_device), 128 ** -0.5
    if block is None:
        loza.loza_ssa_extend(q, k, v, sl, out, lse, ns, win, scale)
    else:
        loza.loza_ssa_extend_blocks(q, k, v, sl, out, lse, ns, win, block, scale)
    G.check(f"extend {c}")
    _all_written(out, "out")
    per = (S + 31) // 32
    perm = torch.randperm(B * per, generator=torch.Generator().manual_seed(8)).to(torch.int32).to(gpu_device)

    def pages(t):
        pool = torch.full((B * per, 32, Hkv, 128), float("nan"), dtype=torch.bfloat16, device=gpu_device)
        for b in range(B):
            rows = torch.full((per * 32, Hkv, 128), float("nan"), dtype=torch.bfloat16, device=gpu_device)
            rows[:S] = t[b]
            pool[perm[b * per:(b + 1) * per].long()] = rows.view(per, 32, Hkv, 128)
        return pool

    k_pool = pages(k)
    o2, l2 = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    fn, pat = (loza.loza_ssa_extend_paged, (ns, win)) if block is None else (loza.loza_ssa_extend_paged_blocks, (ns, win, block))
    fn(q, k_pool, k_pool if alias else pages(v), perm.view(B, per), sl, o2, l2, *pat, scale)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse.view(torch.int32), l2.view(torch.int32))
    for b, L in enumerate(lens):
        first = max(0, q_len - L)
        assert bool((out[b, :first] == 0).all()) and bool(torch.isneginf(lse[b, :, :first]).all())
        full = torch.zeros(1, L, Hq, 128, dtype=torch.bfloat16, device=gpu_device)
        qf, of, lf = full.clone(), full.clone(), torch.zeros(1, Hq, L, device=gpu_device)
        n = q_len - first
        qf[0, L - n:], of[0, L - n:], lf[0, :, L - n:] = q[b, first:], out[b, first:], lse[b, :, first:]
        rows = np.asarray([(h, i) for h in (0, Hq // 2, Hq - 1) for i in range(L - n, L)], dtype=np.int64)
        kb = k[b:b + 1, :L].contiguous()
        H.compare_prefill(qf, kb, kb if alias else v[b:b + 1, :L].contiguous(), of, lf, np.zeros(len(rows), dtype=np.int64),
                          rows[:, 0].copy(), rows[:, 1].copy(), ns, win, scale, f"d128 extend kernel {kernel} L{L}", block)


@pytest.mark.parametrize("kernel,c", [(KERNEL_D128, (1, 1200, 128, 32, False, 128, None, None)), (KERNEL_TILES, (1, 640, 32, 32, False, 128, 300, None))])
@pytest.mark.parametrize("step", ["rise", "jump"])
def test_d128_prefill_scores_that_rise_or_jump(gpu_device, kernel, c, step):
    """Scores that grow by more than the lazy threshold (2^8) every 32 keys, or jump by 2^144 from one key to the
    next: a common direction of queries and keys, its weight a ramp or a step of the position."""
    B, S, Hq, Hkv, _, ns, win, _ = c
    assert _kernel(c) == kernel
    g = torch.Generator(device=gpu_device).manual_seed(80)
    u = torch.randn(128, generator=g, device=gpu_device)
    u = u / u.norm()
    scale = 128 ** -0.5
    i = torch.arange(S, device=gpu_device, dtype=torch.float32)
    level = 0.2 * (i - S / 2) if step == "rise" else torch.where(i < 400, -55.0, 45.0)
    k = (0.3 * torch.randn(B, S, Hkv, 128, generator=g, device=gpu_device) + (level / (scale * 14.0))[None, :, None, None] * u).to(torch.bfloat16)
    q = (0.3 * torch.randn(B, S, Hq, 128, generator=g, device=gpu_device) + 14.0 * u).to(torch.bfloat16)
    v = (0.3 * torch.randn(B, S, Hkv, 128, generator=g, device=gpu_device)).to(torch.bfloat16)   # (small results: once-rounded weights)
    out, lse = H.run_prefill(q, k, v, ns, win, scale)
    assert float(lse[0, 0, S - 1] - lse[0, 0, 200]) > 60.0, "the construction no longer makes the scores rise"
    # (scores of up to +-120: the fp32 log-sum-exp itself is good to half an ulp of that, 4e-6, plus the sum's 2e-5)
    rb, rh, ri = _rows(c)
    ref, ref_lse = H.oracle_prefill_rows(q, k, v, rb, rh, ri, ns, win, scale, 128)
    idx = (torch.as_tensor(rb, device=gpu_device), torch.as_tensor(ri, device=gpu_device), torch.as_tensor(rh, device=gpu_device))
    err = np.abs(out[idx].double().cpu().numpy() - ref)
    assert (err <= H.out_tolerance(ref, torch.bfloat16)).all(), err.max()
    got_lse = lse[torch.as_tensor(rb, device=gpu_device), torch.as_tensor(rh, device=gpu_device), torch.as_tensor(ri, device=gpu_device)]
    assert np.abs(got_lse.double().cpu().numpy() - ref_lse).max() <= 1e-4


@pytest.mark.parametrize("kernel,c", [(KERNEL_D128, (1, 1024, 96, 12, False, 1, 7, 64)), (KERNEL_D128, (1, 1024, 96, 12, True, 1, 7, 64)),
                                      (KERNEL_TILES, (1, 300, 40, 40, False, 1, 2, 64)), (KERNEL_TILES, (1, 300, 40, 40, True, 1, 2, 64))])
def test_d128_calibration(gpu_device, kernel, c):
    """The fp32-output form of both kernels, for the full and the sparse pass."""
    from tests import test_gpu_parity_calibration as C
    B, S, Hq, Hkv, alias, s, l, b = c
    assert _kernel(c) == kernel and _kernel((B, S, Hq, Hkv, alias, 0, None, None)) == kernel
    q, k, v = _inputs(c, gpu_device)
    scale = 128 ** -0.5
    res = C._run(q, k, v, s, l, b, 0.6, scale, 128)
    C._compare(q, k, v, res, *_rows(c), s, l, b, 0.6, scale, f"calib kernel {kernel} {c}")
    full, sparse = H.run_prefill(q, k, v, 0, None, scale, d_v=128), H.run_prefill(q, k, v, s, l, scale, d_v=128, block=b)
    assert torch.equal(res[1].view(torch.int16), full[0].view(torch.int16)) and torch.equal(res[2].view(torch.int16), sparse[0].view(torch.int16))


@pytest.mark.parametrize("kernel,c", [(KERNEL_D128, (1, 517, 192, 24, False, 37, 500, None)), (KERNEL_TILES, (1, 333, 40, 40, True, 5, 100, None))])
def test_d128_prefill_stays_inside_its_buffers(gpu_device, kernel, c):
    B, S, Hq, Hkv, alias, ns, win, _ = c
    assert _kernel(c) == kernel
    q, k, v = _inputs(c, gpu_device)
    G = Guarded(gpu_device)
    out, lse = G.tensor((B, S, Hq, 128), torch.bfloat16), G.tensor((B, Hq, S), torch.float32)
    loza.loza_ssa_prefill(q, k, v, out, lse, ns, win, 128 ** -0.5)
    G.check(f"prefill {c}")
    _all_written(out, "out")
    _all_written(lse, "lse")
