"""Positions around 2^30: a paged cache whose table names the same few pages over and over, so that a long sequence
needs no memory. With a window and no sink the result depends on the window's keys only, and a short sequence whose
table repeats the same pages has the same ones."""
import pytest
import torch

import paper_2512_23966_amd as loza

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,Hq,Hkv,q_len,win", [(128, 96, 24, 512, 400), (128, 32, 8, 40, 400), (128, 80, 20, 400, 90), (576, 64, 1, 200, 300)])
def test_extend(gpu_device, d, Hq, Hkv, q_len, win):
    page, n_pages, d_v = 1024, 3, 512 if d == 576 else 128
    g = torch.Generator(device=gpu_device).manual_seed(9)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, k = r(1, q_len, Hq, d), r(n_pages, page, Hkv, d)
    v = k if d == 576 else r(n_pages, page, Hkv, d)
    long = 2 ** 30 + 200
    res = []
    for L in (long % (n_pages * page) + 5 * n_pages * page, long):
        table = (torch.arange((L + page - 1) // page, device=gpu_device) % n_pages).to(torch.int32).view(1, -1)
        out = torch.full((1, q_len, Hq, d_v), float("nan"), dtype=torch.bfloat16, device=gpu_device)
        lse = torch.full((1, Hq, q_len), float("nan"), dtype=torch.float32, device=gpu_device)
        loza.loza_ssa_extend_paged(q, k, v, table, torch.tensor([L], dtype=torch.int32, device=gpu_device), out, lse, 0, win, d ** -0.5)
        torch.cuda.synchronize()
        res.append((out.float(), lse))
    # two results of the same sums in another order of tiles: each log-sum-exp good to 2e-5, each output to its rounding
    assert float((res[0][1] - res[1][1]).abs().max()) <= 4e-5
    assert float((res[0][0] - res[1][0]).abs().max()) <= 2e-2
