"""Which kernels a call runs, on the host: the rules' edges, and that no plan exceeds what its workspace is sized for."""
import pytest

import paper_2512_23966_amd as loza
from paper_2512_23966_amd import KERNEL_D128, KERNEL_ROWS, KERNEL_TILES


def test_few_rows_are_at_most_512_groups_of_16():
    f = loza.loza_ssa_forward_kernel
    assert f(1, 64, 1, 128, 5000, 576, 128, 1024) == KERNEL_ROWS
    assert f(1, 64, 1, 129, 5000, 576, 128, 1024) == KERNEL_TILES
    assert f(4, 32, 32, 64, 5000, 128, 128, 4096) == KERNEL_ROWS
    assert f(1, 32, 32, 4096, 4096, 128, 128, 4096) == KERNEL_D128


# us with tiles of 256 and of 128 rows; the line was fitted to an earlier kernel of 256 rows and keeps the smaller ones longer
@pytest.mark.parametrize("B,Hq,Hkv,queries,S,sink,local,block,kernel", [
    (1, 32, 32, 8192, 8192, 16, 256, 1, KERNEL_TILES),      # 109, 137: a short window, every head its own keys
    (1, 32, 32, 8192, 8192, 128, 4096, 1, KERNEL_D128),     # 484, 606
    (1, 32, 8, 8192, 8192, 16, 256, 1, KERNEL_D128),        # 77, 97
    (1, 32, 8, 8192, 8192, 1, 7, 128, KERNEL_D128),         # 158, 200
    (1, 32, 32, 4100, 4100, 1, 7, 128, KERNEL_TILES),       # 90, 105: two tiles a head beyond two rounds
    (1, 32, 32, 4100, 4100, 128, 4096, 1, KERNEL_D128),     # 213, 253
    (4, 32, 32, 520, 8192, 16, 256, 1, KERNEL_TILES),       # 52, 61
    (3, 32, 32, 622, 8192, 1, 7, 128, KERNEL_TILES),        # 83, 65: two rounds and one
    (1, 32, 32, 1100, 1100, 128, 4096, 1, KERNEL_TILES),    # 37, 45: 160 tiles
    (8, 32, 32, 300, 8192, 128, 4096, 1, KERNEL_TILES),     # 338, 392: mostly padding
    (1, 32, 8, 6000, 6000, 20, 100, 1, KERNEL_TILES),       # 120 live keys: two-term weights
    (1, 64, 16, 6000, 6000, 0, 1, 300, KERNEL_TILES),       # the first query of a block has one
    (1, 64, 16, 6000, 6000, 1, 3, 64, KERNEL_D128),         # 96, 129
])
def test_width_128_tile_size_by_the_time_model(B, Hq, Hkv, queries, S, sink, local, block, kernel):
    assert loza.loza_ssa_forward_kernel(B, Hq, Hkv, queries, S, 128, sink, local, block) == kernel


@pytest.mark.parametrize("d", [128, 576])
@pytest.mark.parametrize("Hq,Hkv", [(64, 1), (32, 8), (128, 1), (6, 6)])
@pytest.mark.parametrize("sink,local,block", [(128, 8192, 1), (1, 7, 128), (0, 1, 1), (5, None, 1)])
def test_decode_plans_fit_their_workspace(d, Hq, Hkv, sink, local, block):
    for B in (1, 2, 7, 40, 64, 129, 300):
        for S in (1, 64, 5000, 262144):
            kernel, n = loza.loza_ssa_decode_kernel(B, Hq, Hkv, S, d, sink, local, block)
            assert kernel in (KERNEL_ROWS, KERNEL_TILES)
            assert 1 <= n <= loza.loza_ssa_decode_num_splits(B, Hq, Hkv, S, sink * block, None if local is None else local * block)


# (at width 576: the kernels that keep no weights in memory, which take a call whose workspace does not hold them)
@pytest.mark.parametrize("Hq,Hkv,d,S,sink,local,block,split", [
    (64, 1, 576, 16384, 1, 7, 128, (30, 8, 256)),           # backward 12.9 ms whole, 10.5 in chunks
    (64, 1, 576, 16384, 128, 8192, 1, (0, 1, 258)),         # 53.1 whole (the last items are short), 56.8 in chunks
    (64, 1, 576, 14000, 128, 2048, 1, (0, 1, 231)),         # 14.6 and 16.6: 231 items nearly fill the chip
    (64, 1, 576, 8000, 128, 2048, 1, (123, 2, 16)),         # 11.2 and 8.2
    (32, 8, 128, 5000, 0, 2500, 1, (0, 1, 632)),            # 0.79 and 0.84: two workgroups a compute unit
    (32, 1, 128, 8000, 128, 1024, 1, (123, 2, 30)),         # 1.48 and 1.11
])
def test_backward_key_tiles_are_cut_where_that_ends_sooner(Hq, Hkv, d, S, sink, local, block, split):
    d_v, shared = (512, True) if d == 576 else (128, False)
    assert loza.loza_ssa_backward_split(1, Hq, Hkv, S, d, d_v, sink, local, block, shared) == split


@pytest.mark.parametrize("B,Hq,Hkv,d,S,sink,local,kernel", [
    (130, 48, 1, 576, 16384, 128, 8192, KERNEL_TILES),      # 341 against 403 us of the few-rows kernel
    (64, 48, 1, 576, 16384, 128, 2048, KERNEL_TILES),       # 54 against 59
    (8, 64, 1, 576, 16384, 128, 2048, KERNEL_ROWS),         # 38 against 22
    (8, 64, 1, 576, 16384, 128, 8192, KERNEL_ROWS),         # 50 against 40
    (16, 64, 1, 576, 16384, 128, 8192, KERNEL_TILES),       # 56 against 65
    (64, 64, 1, 576, 262144, 128, 8192, KERNEL_TILES),
    (300, 32, 1, 576, 16384, 128, 8192, KERNEL_ROWS),       # at most two groups of 16 heads
])
def test_decode_kernel_by_size(B, Hq, Hkv, d, S, sink, local, kernel):
    assert loza.loza_ssa_decode_kernel(B, Hq, Hkv, S, d, sink, local)[0] == kernel


@pytest.mark.parametrize("Hkv,pattern", [(8, (128, 4096, 1)), (32, (128, 4096, 1)), (1, (128, 8192, 1)), (8, (1, 7, 128)), (16, (128, 32000, 1))])
def test_extends_of_the_larger_tiles_take_no_scratch_memory(Hkv, pattern):
    """3 sequences of 385 tokens, 8 key heads, 128 + 4096: 130 us, as three parts of the smaller tiles 212."""
    larger = 0
    for B in (1, 2, 3, 6, 7, 8, 16):
        for q_len in (*range(100, 700, 3), 1283, 1300):
            if loza.loza_ssa_forward_kernel(B, 32, Hkv, q_len, 65536, 128, *pattern) == KERNEL_D128:
                larger += 1
                assert loza.loza_ssa_extend_workspace_bytes(B, 32, Hkv, 65536, q_len, 128, 128, *pattern) == 0, (B, q_len)
    assert larger > 50


def test_refused_sizes():
    for call in (lambda: loza.loza_ssa_forward_kernel(1, 3, 2, 8, 8, 128, 0, 1), lambda: loza.loza_ssa_forward_kernel(1, 2, 2, 9, 8, 128, 0, 1),
                 lambda: loza.loza_ssa_decode_kernel(1, 2, 2, 8, 64, 0, 1), lambda: loza.loza_ssa_decode_kernel(0, 2, 2, 8, 128, 0, 1),
                 lambda: loza.loza_ssa_backward_split(1, 96, 1, 8, 64, 64, 0, 1), lambda: loza.loza_ssa_backward_split(1, 2, 1, 8, 128, 128, 0, 0)):
        with pytest.raises(loza.LozaError):
            call()
