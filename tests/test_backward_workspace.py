"""What the workspace of the absorbed-MLA backward holds, on the host."""
import pytest

import paper_2512_23966_amd as loza

GIB = 1 << 30


def _bytes(B, S, Hq, Hkv, pattern):
    """(all of it, the row statistics)"""
    return loza.loza_ssa_backward_workspace_bytes_blocks(B, Hq, Hkv, S, 576, 512, *pattern, True), B * Hkv * ((S * Hq // Hkv + 31) // 32 * 32) * 8


@pytest.mark.parametrize("Hq", [16, 64, 128])
@pytest.mark.parametrize("pattern", [(1, 7, 128), (128, 8192, 1), (16, 256, 1)])
def test_long_sequences_take_what_their_windows_need(Hq, pattern):
    """Sums that go on from a chunk of rows to the next are those of the groups of keys that rows on both sides see."""
    for S in (131072, 1 << 20, 1 << 22):
        n, stat = _bytes(1, S, Hq, 1, pattern)
        assert 0 < n - stat < 2.5 * GIB


@pytest.mark.parametrize("B,S,Hq,pattern,slots,chunk_tiles", [
    (1, 2048, 64, (1, 7, 128), 10, 1024),            # a sink group, and nine that 1 + 7 blocks of 128 can touch
    (2, 1000, 16, (0, 300, 1), 4, 125),              # two sequences in a chunk
    (1, 131072, 64, (128, 8192, 1), 67, 256),        # chunks of 256 row tiles
])
def test_what_it_is_made_of(B, S, Hq, pattern, slots, chunk_tiles):
    """4 bytes a pair of 128 rows x 128 keys, then whole partial results of 128 keys x 576 (and of the sums between chunks)."""
    n, stat = _bytes(B, S, Hq, 1, pattern)
    rest = n - stat - B * chunk_tiles * slots * 128 * 128 * 4
    assert rest > 0 and rest % (128 * 576 * 4) == 0 and rest < 0.5 * GIB


@pytest.mark.parametrize("B,S,Hq,pattern,given_out", [
    (1, 3000, 64, (0, 3000, 1), 2092756992),
    (1, 8000, 64, (128, 4096, 1), 1858797568),
    (1, 16384, 64, (1, 7, 128), 2209906688),
])
def test_sizes_that_callers_may_have_kept_are_enough(B, S, Hq, pattern, given_out):
    """(given out while every group of keys had a place for sums between chunks of rows)"""
    assert _bytes(B, S, Hq, 1, pattern)[0] <= given_out
