"""Backward of the absorbed-MLA shape through weights in memory: against the kernels that keep none, which take a call
whose workspace does not hold them (the other backward tests compare both with the oracle, at forms of their own). Edges: rows
and keys that end inside a tile, row tiles that straddle positions, groups of keys that only some rows of a segment
see, sinks that end inside a group or meet the window, rows in several chunks, several (sequence, key head)s in one."""
import pytest
import torch

import paper_2512_23966_amd as loza


@pytest.mark.gpu
@pytest.mark.parametrize("B,S,Hq,Hkv,sink,local,block", [
    (1, 1, 64, 1, 0, 1, 1),             # one position: half a row tile
    (1, 127, 64, 1, 5, 40, 1),
    (1, 129, 64, 1, 0, 129, 1),         # every key live, one key in the second group
    (2, 300, 32, 1, 130, 70, 1),        # sinks end inside a group; two sequences in a chunk
    (1, 700, 64, 2, 1, 2, 128),         # two key heads
    (1, 513, 128, 1, 20, 200, 1),       # a row tile is one position
    (1, 500, 96, 1, 2, 3, 37),          # row tiles that straddle positions unevenly, blocks of no round size
    (1, 900, 8, 1, 128, 300, 1),        # a row tile is 16 positions
    (1, 2000, 2, 1, 0, 500, 1),         # a row tile is 64 positions
    (3, 700, 64, 1, 1, 3, 64),
    (1, 3000, 64, 1, 0, 3000, 1),       # two chunks of rows, every key seen by both
    (1, 7000, 64, 1, 1, 7, 128),        # three chunks, a window that leaves the first keys behind
    (2, 2600, 64, 1, 100, 1800, 1),     # chunks of one sequence after the other
])
def test_weights_in_memory_against_none(gpu_device, B, S, Hq, Hkv, sink, local, block):
    g = torch.Generator(device=gpu_device).manual_seed(S + Hq)
    r = lambda *s: torch.randn(*s, generator=g, device=gpu_device).to(torch.bfloat16)
    q, k, dout = r(B, S, Hq, 576), r(B, S, Hkv, 576), r(B, S, Hq, 512)
    out, lse, scale = torch.empty_like(dout), torch.empty(B, Hq, S, device=gpu_device), 192 ** -0.5
    loza.loza_ssa_prefill_blocks(q, k, k, out, lse, sink, local, block, scale)
    n = loza.loza_ssa_backward_workspace_bytes_blocks(B, Hq, Hkv, S, 576, 512, sink, local, block, True)
    rows = B * Hkv * ((S * Hq // Hkv + 31) // 32 * 32)
    assert n > rows * (8 + 2 * 2 * 32)                      # statistics, and weights of more than 32 keys
    got = []
    for size in (n, n, n - 1):
        dq, dk = torch.full_like(q, float("nan")), torch.full_like(k, float("nan"))
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=gpu_device)   # NaNs: nothing is read that was not written
        loza.loza_ssa_backward_blocks(q, k, k, out, lse, dout, dq, dk, None, sink, local, block, scale, ws)
        got.append((dq, dk))
    for a, b, c in zip(*got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        # Same operands and the same single rounding of p and dS; sums in another order may round a result to its neighbour,
        # one step of bf16 (at most 2^-7 of the value) away, and a weight to its own, which moves a sum by
        # far less than four of the gradient bound's units (2^-9 of the row's rms).
        a, c = a.float(), c.float()
        rms = c.pow(2).mean(-1, keepdim=True).sqrt()
        assert bool(((a - c).abs() <= 2.0 ** -7 * (rms + c.abs()) + 2e-5).all()), float(((a - c).abs() / (rms + 1e-9)).max())


def test_which_calls_keep_weights():
    def bytes_per_row(B, S, local, block=1, Hq=64):
        return loza.loza_ssa_backward_workspace_bytes_blocks(B, Hq, 1, S, 576, 512, 0, local, block, True) / (B * S * Hq)
    assert bytes_per_row(1, 1024, 128) > 100 and bytes_per_row(1, 1026, 128) == 8 and bytes_per_row(1, 1026, 129) > 100
    assert bytes_per_row(4, 1000, 500, Hq=4) > 100 and bytes_per_row(5, 1000, 500, Hq=4) == 8   # key heads against query heads a group
    assert bytes_per_row(8, 128, 128) > 100 and bytes_per_row(9, 128, 128) == 8 and bytes_per_row(9, 129, 129) > 100


@pytest.mark.parametrize("B,S,Hq,pattern,weights", [
    (1, 11988, 2, (0, 200, 1), False), (1, 64000, 2, (128, 2048, 1), True),     # us without and with: 109, 134; 2174, 1860
    (3, 8653, 4, (0, 200, 1), False), (1, 8000, 4, (1, 7, 128), True),          # 375, 440; 380, 281
    (8, 12201, 8, (0, 256, 1), False), (1, 8000, 8, (1, 7, 128), True),         # 2725, 2885; 731, 486
    (16, 500, 8, (1, 7, 128), True), (16, 786, 8, (0, 200, 1), False),          # 280, 290 (what the line costs); 321, 370
    (1, 4096, 4, (0, 200, 1), True), (1, 4097, 4, (0, 200, 1), False),          # 4,096 keys leave most of the chip idle
    (2, 4096, 4, (16, 320, 1), True), (2, 4097, 4, (16, 320, 1), False),        # with sink keys twice as many
    (1, 6500, 2, (1, 7, 128), False),                                           # 200, 234
])
def test_few_heads_a_group_and_short_windows_keep_none(B, S, Hq, pattern, weights):
    n = loza.loza_ssa_backward_workspace_bytes_blocks(B, Hq, 1, S, 576, 512, *pattern, True)
    assert (n > B * S * Hq * 1000) == weights
