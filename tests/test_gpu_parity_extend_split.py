"""Extends whose keys several workgroups share (scratch memory for their partial results): both kernels that split, at
the edges of what they handle, against the oracle; the rows that must not come from once-rounded weights; scratch
memory given or not, too small, on another stream and under capture."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2512_23966_amd as loza
from paper_2512_23966_amd import binding as B_
from tests import helpers as H
from tests.test_gpu_parity_extend import _rand, _run, _run_paged

FAKE = 4096


def _plan(B, Hq, Hkv, S_max, q_len, d, ns, win, block=1):
    """Sets of partial results per row (1: none)."""
    d_v = 512 if d == 576 else 128
    return loza.loza_ssa_extend_workspace_bytes(B, Hq, Hkv, S_max, q_len, d, d_v, ns, win, block) // (B * Hq * q_len * (d_v + 4) * 4) or 1


def _check(q, kc, vc, lens, out, lse, pattern, scale, label, block=None, step=1):
    """Every `step`-th row (b, r, h) of a position >= 0 against the oracle; the others must be 0 / -inf."""
    B, q_len, Hq, _ = q.shape
    rows = [(b, r, h) for b, L in enumerate(lens) for r in range(q_len) if L - q_len + r >= 0 for h in range(Hq)][::step]
    for b, L in enumerate(lens):
        dead = max(0, q_len - L)
        assert (out[b, :dead] == 0).all() and torch.isneginf(lse[b, :, :dead]).all(), f"{label}: queries before the start"
    rb, rr, rh = (np.asarray(x, dtype=np.int64) for x in zip(*rows))
    ri = np.asarray(lens, dtype=np.int64)[rb] - q_len + rr
    tb, tr, th = (torch.as_tensor(x, device=q.device) for x in (rb, rr, rh))
    ref_out, ref_lse = oracle.ssa_rows(q[tb, tr, th].contiguous().cpu(), kc.cpu(), ("alias", out.shape[3]) if vc is kc else vc.cpu(), rb, rh, ri,
                                       Hq=Hq, n_sink=pattern[0], window=pattern[1], scale=scale, block=block)
    H._judge(out[tb, tr, th].double().cpu().numpy(), ref_out, lse[tb, th, tr].double().cpu().numpy(), ref_lse, torch.bfloat16, len(rb), label)


# B, Hq, Hkv, d, S_max, q_len, lens, n_sink, window, block, page, rows of the oracle
CASES = [
    (1, 64, 1, 576, 2600, 1, [2600], 128, 2048, None, 0, 1),             # one token: splits of a tile or two a wave
    (3, 64, 1, 576, 2560, 4, [2509, 131, 2], 128, 1500, None, 128, 1),   # around position 128; queries before the start
    (2, 64, 1, 576, 3000, 11, [2999, 0], 1, 20, 128, 0, 1),              # blocks; an empty cache; rows no multiple of 16
    (1, 128, 2, 576, 2048, 3, [2047], 0, 1200, None, 32, 1),             # two latents
    (2, 8, 2, 128, 4000, 5, [4000, 77], 70, 3000, None, 0, 1),           # separate values, 4 heads a group
    (1, 6, 2, 128, 2048, 19, [2011], 16, 1500, None, 64, 1),             # 3 heads a group
    (4, 64, 1, 576, 6144, 33, [6143, 5001, 150, 20], 128, 5000, None, 0, 23),  # the tile kernel; tiles among the first positions
    (2, 64, 1, 576, 8192, 65, [8192, 7001], 0, 7000, None, 128, 29),     # odd number of positions: half a tile at the end
    (4, 32, 8, 128, 2304, 70, [2304, 2111, 150, 64], 64, 2000, None, 0, 29),   # narrow tiles, separate values
]


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,S_max,q_len,lens,ns,win,block,page,step", CASES)
def test_split_extend(gpu_device, B, Hq, Hkv, d, S_max, q_len, lens, ns, win, block, page, step):
    n = _plan(B, Hq, Hkv, S_max, q_len, d, ns, win, block or 1)
    assert n > 1
    q, kc = _rand((B, q_len, Hq, d), 61, torch.bfloat16, gpu_device), _rand((B, S_max, Hkv, d), 62, torch.bfloat16, gpu_device)
    vc = kc if d == 576 else _rand((B, S_max, Hkv, d), 63, torch.bfloat16, gpu_device)
    for b, L in enumerate(lens):
        kc[b, L:] = float("nan")
        vc[b, L:] = float("nan")
    seqlens, scale, d_v = torch.tensor(lens, dtype=torch.int32, device=gpu_device), (192 if d == 576 else 128) ** -0.5, 512 if d == 576 else 128
    if page:
        from tests.test_gpu_parity_paged import _paginate
        pages, table = _paginate(kc, lens, page, seed=3)
        vpages = pages if vc is kc else _paginate(vc, lens, page, seed=3)[0]
        out, lse = _run_paged(q, pages, vpages, table, seqlens, (ns, win), scale, d_v, block)
    else:
        out, lse = _run(q, kc, vc, seqlens, (ns, win), scale, d_v, block)
    _check(q, kc, vc, lens, out, lse, (ns, win), scale, f"split {n}: q{q_len} lens{lens} ns{ns} W{win} b{block}", block, step)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,S_max,q_len,ns,win", [(2, 8, 2, 4000, 5, 70, 3000), (4, 32, 8, 2304, 70, 64, 2000)])   # few rows; tiles
def test_split_extend_d128_values_are_the_keys(gpu_device, B, Hq, Hkv, S_max, q_len, ns, win):
    assert _plan(B, Hq, Hkv, S_max, q_len, 128, ns, win) > 1
    lens, scale = [S_max, q_len - 2, 150, S_max - 77][:B], 128 ** -0.5
    q, kc = _rand((B, q_len, Hq, 128), 69, torch.bfloat16, gpu_device), _rand((B, S_max, Hkv, 128), 70, torch.bfloat16, gpu_device)
    for b, L in enumerate(lens):
        kc[b, L:] = float("nan")
    out, lse = _run(q, kc, kc, torch.tensor(lens, dtype=torch.int32, device=gpu_device), (ns, win), scale, 128)
    _check(q, kc, kc, lens, out, lse, (ns, win), scale, f"split, d128 aliased: q{q_len}", None, 13)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [576, 128])
def test_large_results_do_not_come_from_split_tiles(gpu_device, d):
    """Rows whose weight sits on one key, in some groups of 16 rows and not in others."""
    B, Hq, Hkv, S_max, q_len = (4, 64, 1, 6144, 33) if d == 576 else (4, 32, 8, 2304, 70)
    ns, win, lens = 16, 5000 if d == 576 else 2000, [S_max, S_max - 7, S_max - 500, S_max - 1001]
    assert _plan(B, Hq, Hkv, S_max, q_len, d, ns, win) > 1
    q, kc = _rand((B, q_len, Hq, d), 64, torch.bfloat16, gpu_device), _rand((B, S_max, Hkv, d), 65, torch.bfloat16, gpu_device)
    vc = kc if d == 576 else _rand((B, S_max, Hkv, d), 66, torch.bfloat16, gpu_device)
    q[0, 3, 5] = 2 * kc[0, S_max - 100, 5 * Hkv // Hq]      # its weight sits on that key
    q[2] *= 4
    seqlens, scale, d_v = torch.tensor(lens, dtype=torch.int32, device=gpu_device), (192 if d == 576 else 128) ** -0.5, 512 if d == 576 else 128
    out, lse = _run(q, kc, vc, seqlens, (ns, win), scale, d_v)
    assert out[0, 3, 5].abs().max() >= 2
    _check(q, kc, vc, lens, out, lse, (ns, win), scale, f"large results d{d}", None, 17)
    k0 = kc[:1]
    _check(q[:1, 3:4], k0, k0 if vc is kc else vc[:1], [S_max - q_len + 4], out[:1, 3:4], lse[:1, :, 3:4], (ns, win), scale, f"peaked row d{d}")


@pytest.mark.gpu
def test_scratch_memory(gpu_device):
    B, Hq, S_max, q_len, lens, pat, scale = 2, 64, 3000, 5, [3000, 1234], (128, 2000), 192 ** -0.5
    q, kc = _rand((B, q_len, Hq, 576), 67, torch.bfloat16, gpu_device), _rand((B, S_max, 1, 576), 68, torch.bfloat16, gpu_device)
    seqlens = torch.tensor(lens, dtype=torch.int32, device=gpu_device)
    need = loza.loza_ssa_extend_workspace_bytes(B, Hq, 1, S_max, q_len, 576, 512, *pat)
    assert need > 0
    same = lambda a, b: all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b))
    fresh = lambda: (torch.full((B, q_len, Hq, 512), float("nan"), dtype=torch.bfloat16, device=gpu_device),
                     torch.full((B, Hq, q_len), float("nan"), device=gpu_device))
    call = lambda o, **kw: loza.loza_ssa_extend(q, kc, kc, seqlens, *o, *pat, scale, **kw)
    ref = fresh()
    call(ref)
    torch.cuda.synchronize()
    # a workspace of the caller's, between guard bytes, with anything in it
    ws = torch.full((need + 512,), 255, dtype=torch.uint8, device=gpu_device)
    got = fresh()
    call(got, workspace=ws[256:256 + need])
    torch.cuda.synchronize()
    assert same(got, ref) and (ws[:256] == 255).all() and (ws[256 + need:] == 255).all()
    with pytest.raises(loza.LozaError) as e:
        call(got, workspace=ws[256:256 + need - 1])
    assert e.value.status == -4
    # another stream, by object and by handle
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (side, side.cuda_stream):
        got = fresh()
        torch.cuda.synchronize()
        call(got, stream=stream)
        side.synchronize()
        assert same(got, ref)
    # under capture: without scratch memory of the caller's the launches without it, with it the same as above
    whole = fresh()
    L = B_.lib()
    assert L.loza_ssa_extend(q.data_ptr(), kc.data_ptr(), kc.data_ptr(), seqlens.data_ptr(), whole[0].data_ptr(), whole[1].data_ptr(), B, Hq, 1,
                             S_max, q_len, 576, 512, *pat, scale, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    for kw, want in (({}, whole), ({"workspace": ws[256:256 + need]}, ref)):
        got = fresh()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(got, **kw)
        for _ in range(3):
            got[0].zero_()
            torch.randn(1 << 20, device=gpu_device).sum().item()
            graph.replay()
            torch.cuda.synchronize()
            assert same(got, want)


def test_what_splits_and_what_does_not():
    assert _plan(1, 64, 1, 65536, 2, 576, 128, 8192) >= 16
    assert _plan(16, 64, 1, 65536, 4, 576, 128, 8192) == 1            # 256 groups of 16 rows: a round of the few-rows kernel
    assert _plan(4, 64, 1, 65536, 36, 576, 128, 8192) >= 2            # the tile kernel
    assert _plan(4, 64, 1, 65536, 1000, 576, 128, 8192) == 1          # fills the chip by itself
    assert _plan(1, 64, 1, 450, 450, 576, 16, 130) == 1               # the whole sequence: a prefill
    # few live keys: what the host and the merge take is more than the split saves
    assert _plan(1, 64, 1, 16384, 28, 576, 1, 7, 128) == 1            # 25.6 us, in two parts 28.5
    assert _plan(9, 64, 1, 16384, 3, 576, 1, 7, 128) == 1             # 25.6 and 28.3
    assert _plan(1, 32, 8, 16384, 4, 128, 1, 7, 128) == 1             # 11.9, in 16 parts 8.6 and 5 of the host
    assert _plan(1, 64, 1, 16384, 2, 576, 1, 7, 128) > 1              # 25.1 and 14.1
    # one round of tiles: where a split costs nothing it is taken, since an unsplit tile may be computed again; the plan
    # does not hang on a single key (parts at 1,020 to 1,300 live keys)
    assert _plan(24, 64, 1, 65536, 6, 576, 1, 7, 128) == 3            # 65 us, 152 with a large result, 62 split
    assert _plan(16, 64, 1, 65536, 13, 576, 1, 7, 128) == 1           # 65, 152, in two parts 71
    assert _plan(16, 64, 1, 65536, 13, 576, 0, 500) == 1              # 43, 99, in two parts 55
    for B, q_len in ((8, 32), (1, 256), (4, 64), (24, 6)):
        plans = [_plan(B, 64, 1, 65536, q_len, 576, 0, w) for w in range(1020, 1300)]
        assert len(set(plans)) == 1
    # rows in two to four parts; tiles in 15 to 33 parts were no faster, and twice as slow where caches are short
    assert _plan(8, 64, 1, 65536, 4, 576, 128, 4096) == 2             # 57 us, as tiles 59; caches of 200 to 400 rows 23 and 37
    assert _plan(7, 64, 1, 65536, 2, 576, 128, 8192) == 4             # 51 and 63; 18 and 43
    for bad in ((0, 64, 1, 100, 2, 576, 512, 1, 9, 1), (1, 64, 1, 100, 101, 576, 512, 1, 9, 1), (1, 64, 1, 100, 2, 577, 512, 1, 9, 1),
                (1, 64, 1, 100, 2, 576, 512, -1, 9, 1), (1, 64, 1, 100, 2, 576, 512, 1, 0, 1), (1, 64, 1, 100, 2, 576, 512, 1, 9, 0)):
        assert loza.loza_ssa_extend_workspace_bytes(*bad) == 0
    for B in (1, 2, 5, 16, 200):                                      # the scratch memory stays below 2 rounds of tiles
        for q_len in (1, 2, 7, 100, 2048):
            for Hq, Hkv, d in ((64, 1, 576), (32, 8, 128), (32, 32, 128), (3, 1, 128)):
                n = _plan(B, Hq, Hkv, 1 << 20, q_len, d, 128, 8192)
                assert 1 <= n <= 64 and (n == 1 or n * B * Hq * q_len <= 1024 * 128 + 128 * n * B * Hkv)


# What these calls needed while their rows, not tiles, shared keys (4 bytes x (512 + 4) x rows x parts; none: one part)
KEPT = [(8, 4, 65536, (128, 8192, 1), 2), (1, 32, 65536, (128, 8192, 1), 2), (2, 8, 65536, (128, 8192, 1), 4)]


@pytest.mark.parametrize("B,q_len,S_max,pattern,parts", KEPT)
def test_the_least_scratch_memory_of_few_rows(B, q_len, S_max, pattern, parts):
    size = 4 * (512 + 4) * B * 64 * q_len * parts

    def call(nbytes, ws=FAKE + 4):                                    # (misaligned: no call gets beyond its argument checks)
        return B_.lib().loza_ssa_extend_with_workspace(FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, B, 64, 1, S_max, 0, 0, 0, q_len, 576, 512, *pattern,
                                                       0.07, ws, nbytes, None)
    assert call(size) == -6 and call(size - 1) == -4 and call(0, None) == -4


@pytest.mark.gpu
@pytest.mark.parametrize("B,q_len,lens,parts", [(2, 16, [6000, 5555], 2), (5, 15, [6000, 5600, 700, 9, 0], 1), (5, 13, [6000, 5999, 140, 18, 2222], 1)])
def test_few_rows_with_little_scratch_memory(gpu_device, B, q_len, lens, parts):
    """A workspace for the few-rows kernel alone, or none where that kernel does not split the call."""
    S_max, pat, scale = 6000, (128, 5000), 192 ** -0.5
    full = loza.loza_ssa_extend_workspace_bytes(B, 64, 1, S_max, q_len, 576, 512, *pat)
    size = 4 * (512 + 4) * B * 64 * q_len * parts if parts > 1 else 0
    assert full > size
    q, kc = _rand((B, q_len, 64, 576), 71, torch.bfloat16, gpu_device), _rand((B, S_max, 1, 576), 72, torch.bfloat16, gpu_device)
    seqlens = torch.tensor(lens, dtype=torch.int32, device=gpu_device)
    ws = torch.full((size + 512,), 255, dtype=torch.uint8, device=gpu_device)
    out = torch.full((B, q_len, 64, 512), float("nan"), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.full((B, 64, q_len), float("nan"), device=gpu_device)
    rc = B_.lib().loza_ssa_extend_with_workspace(q.data_ptr(), kc.data_ptr(), kc.data_ptr(), None, seqlens.data_ptr(), out.data_ptr(), lse.data_ptr(),
                                                 B, 64, 1, S_max, 0, 0, 0, q_len, 576, 512, *pat, 1, scale, ws.data_ptr() + 256 if size else None, size,
                                                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and (ws[:256] == 255).all() and (ws[256 + size:] == 255).all()
    _check(q, kc, kc, lens, out, lse, pat, scale, f"little scratch memory: {B} x {q_len}", None, 17)


def test_bad_arguments_are_rejected_before_any_launch():
    def call(ws=FAKE, nbytes=1 << 40, table=None, seqlens=FAKE, q_len=4, page=64, block=1, scale=0.07):
        return B_.lib().loza_ssa_extend_with_workspace(FAKE, FAKE, FAKE, table, seqlens, FAKE, FAKE, 2, 64, 1, 8192, 256, page, 128, q_len, 576, 512, 128,
                                                       4096, block, scale, ws, nbytes, None)
    assert call(ws=None) == -4 and call(nbytes=1000) == -4 and call(ws=FAKE + 4) == -6
    assert call(seqlens=None) == -1 and call(q_len=0) == -2 and call(block=0) == -2 and call(scale=0.0) == -2
    assert call(table=FAKE, page=48) == -2 and call(table=FAKE + 2) == -6
