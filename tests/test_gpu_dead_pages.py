"""Extend against a paged cache whose pages without a live key are evicted: their table entries are stale (out of
range, or the number of a page of NaN and infinities) and their rows poisoned. A call may read only pages that
hold a key some query of it sees, so the bits must be those of the call on the intact cache."""
import numpy as np
import pytest
import torch

import paper_2512_23966_amd as loza

pytestmark = pytest.mark.gpu


def _live_pages(L, q_len, ns, win, block, page):
    """Logical pages that hold a live key of one of the last q_len positions of L."""
    i = np.arange(max(0, L - q_len), L)
    b = block or 1
    wb = np.maximum(0, i // b - win + 1) * b
    j = np.zeros(L, dtype=bool)
    j[:min(ns * b, L)] = True
    for lo, hi in zip(wb, i):
        j[lo:hi + 1] = True
    return sorted(set((np.nonzero(j)[0] // page).tolist()))


# enough tiles of 256 rows for the kernel that copies 64 keys at a time
@pytest.mark.parametrize("alias", [False, True])
@pytest.mark.parametrize("lens,q_len,Hq,Hkv,ns,win,block,page", [
    ([1500], 512, 96, 24, 32, 400, None, 32),     # the second half of the sink's 64 keys is dead
    ([1500], 512, 96, 24, 0, 380, None, 32),      # so is the first half of the first window tile
    ([1490, 1303], 512, 48, 12, 33, 450, None, 32),
    ([1535], 512, 96, 24, 1, 13, 32, 32),         # block-granular
    ([1700], 509, 96, 24, 70, 600, None, 64),
    ([900], 512, 96, 6, 5, 260, None, 32),
])
def test_d128_extend_reads_only_pages_with_a_live_key(gpu_device, alias, lens, q_len, Hq, Hkv, ns, win, block, page):
    B = len(lens)
    cap = (max(lens) + page - 1) // page * page
    assert loza.loza_ssa_forward_kernel(B, Hq, Hkv, q_len, cap, 128, ns, win, block or 1) == loza.KERNEL_D128
    g = torch.Generator(device=gpu_device).manual_seed(61)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    max_pages = (max(lens) + page - 1) // page
    num = B * max_pages + 1                                  # page 0: what a stale entry leads to
    q, kp = r(B, q_len, Hq, 128), r(num, page, Hkv, 128)
    vp = kp if alias else r(num, page, Hkv, 128)
    table = 1 + torch.randperm(B * max_pages, generator=torch.Generator().manual_seed(3)).to(torch.int32).view(B, max_pages)
    scale = 128 ** -0.5

    def run(k, v, t):
        out = torch.full((B, q_len, Hq, 128), float("nan"), dtype=torch.bfloat16, device=gpu_device)
        lse = torch.full((B, Hq, q_len), float("nan"), dtype=torch.float32, device=gpu_device)
        sl = torch.tensor(lens, dtype=torch.int32, device=gpu_device)
        fn, pat = (loza.loza_ssa_extend_paged, (ns, win)) if block is None else (loza.loza_ssa_extend_paged_blocks, (ns, win, block))
        fn(q, k, v, t.to(gpu_device), sl, out, lse, *pat, scale)
        torch.cuda.synchronize()
        return out, lse

    clean = run(kp, vp, table)
    bad = torch.tensor([0] + [int(table[b, p]) for b in range(B) for p in range(max_pages)
                              if p not in _live_pages(lens[b], q_len, ns, win, block, page)], device=gpu_device)
    kb = kp.clone()
    kb[bad], kb[bad, 1::2] = float("nan"), float("inf")
    vb = kb if alias else vp.clone()
    vb[bad], vb[bad, ::2] = float("inf"), float("nan")
    stale = table.clone()
    for b in range(B):
        dead = [p for p in range(max_pages) if p not in _live_pages(lens[b], q_len, ns, win, block, page)]
        stale[b, dead[::2]] = -7                             # leads to page 0
    for t in (table, stale):
        out, lse = run(kb, vb, t)
        assert bool(torch.isfinite(out.float()).all()), "a page without a live key was read"
        assert torch.equal(out.view(torch.int16), clean[0].view(torch.int16)) and torch.equal(lse, clean[1])
