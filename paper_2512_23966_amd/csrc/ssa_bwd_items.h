// Work items of the key-stationary backward kernels (device side).
#ifndef LOZA_SSA_BWD_ITEMS_H
#define LOZA_SSA_BWD_ITEMS_H

#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

// One workgroup's share: the row tiles [yt_begin, yt_begin + nt) that can see keys [64 xt, 64 xt + 64) of batch b,
// key head g, walked from yt_start around. partial: they are a chunk of the rows that see those keys, and the results
// go to tile `slot` of the fp32 partial sums. nt <= 0: nothing (a chunk beyond the rows of its key tile).
struct BwdItem {
    int b, g, xt;
    int yt_begin, yt_start, nt;
    bool partial;
    int64_t slot;
};

static __device__ __forceinline__ BwdItem bwd_key_item(const BwdParams &p, const int workgroup)
{
    const int n_kt = (int)((p.S + 63) / 64);
    int b, g, xt, chunk = 0;
    bool partial = false;    // leave an fp32 partial sum for the reduce kernel
    bool is_split = false;   // a chunk of a key tile that is split for balance
    const int kt0 = p.max_chunks > 1 ? p.n_sink_kt : 0;               // key tiles before it run in chunks
    const int items = kt0 * p.max_chunks + (n_kt - kt0 - p.n_split_kt), BH = p.B * p.Hkv;
    // Workgroups go to the eight XCDs round-robin and every XCD has an L2 of its own. Handing every
    // XCD one contiguous eighth of the items makes the workgroups that share an L2 neighbouring key
    // tiles, whose row ranges overlap almost completely (see the rotation below). The chunks of split
    // tiles come last, dealt out the same way among themselves.
    auto per_xcd = [](int id, int total) {
        const int eighth = total / 8;
        return id < eighth * 8 ? (id % 8) * eighth + id / 8 : id;
    };
    int id = workgroup;
    is_split = id >= items * BH;
    int it, per;
    if (!is_split) {
        id = per_xcd(id, items * BH);
        per = items;
    } else {
        per = p.n_split_kt * p.split_chunks;
        id = per_xcd(id - items * BH, per * BH);
    }
    it = id % per;
    id /= per;
    g = id % p.Hkv;
    b = id / p.Hkv;
    if (is_split) {
        xt = kt0 + it / p.split_chunks;
        chunk = it % p.split_chunks;
        partial = true;
    } else if (it < kt0 * p.max_chunks) {
        xt = it / p.max_chunks;
        chunk = it % p.max_chunks;
        partial = true;
    } else {
        xt = kt0 + p.n_split_kt + (it - kt0 * p.max_chunks);
    }

    int yt_lo, yt_hi;
    bwd_key_tile_rows(p, xt, yt_lo, yt_hi);
    int yt_begin = yt_lo;
    int yt_end = yt_hi + 1;
    if (partial) {
        const int ct = is_split ? (yt_end - yt_lo + p.split_chunks - 1) / p.split_chunks : p.chunk_tiles;
        yt_begin = yt_lo + chunk * ct;
        if (yt_begin + ct < yt_end) yt_end = yt_begin + ct;
    }
    const int nt = yt_end - yt_begin;
    // Neighbouring key tiles see almost the same rows, each range shifted by 64 positions. Left to
    // start at its own first row tile, every workgroup would stream its q and dout rows at a
    // different place at any moment, and all of it would come from HBM (at the 128K shape: 2.4 TB
    // per launch). Instead the 32 key tiles of a group (the workgroups that run together on one
    // XCD) all start at the first row tile of the group's last member and wrap around inside their
    // own range: they then ask for the same row tile at about the same time, and one fetch into
    // the shared L2 serves all of them.
    int yt_start = yt_begin;
    if (xt >= p.n_sink_kt && !is_split) {
        const int k0 = p.max_chunks > 1 || p.n_split_kt > p.n_sink_kt ? p.split_kt0() + p.n_split_kt : p.n_sink_kt;
        const int last = k0 + ((xt - k0) / 32) * 32 + 31;
        int a_lo, a_hi;
        bwd_key_tile_rows(p, last < n_kt - 1 ? last : n_kt - 1, a_lo, a_hi);
        if (a_lo >= yt_begin && a_lo < yt_end) yt_start = a_lo;
    } else if (is_split) {
        // (an XCD runs all chunks of 32 / split_chunks key tiles at a time: those of equal number go together,
        // unless chunks are so short that the tiles' own shift has them start where other chunks do)
        const int kt0 = p.split_kt0(), grp = p.split_chunks < 32 ? 32 / p.split_chunks : 1, end = kt0 + p.n_split_kt - 1;
        const int first = kt0 + ((xt - kt0) / grp) * grp, last = first + grp - 1 < end ? first + grp - 1 : end;
        int f_lo, a_lo, a_hi;
        bwd_key_tile_rows(p, first, f_lo, a_hi);
        bwd_key_tile_rows(p, last, a_lo, a_hi);
        const int ct = (a_hi - a_lo + p.split_chunks) / p.split_chunks, start = a_lo + chunk * ct;
        if (a_lo - f_lo < ct && start >= yt_begin && start < yt_end) yt_start = start;
    }
    const int64_t bg = (int64_t)b * p.Hkv + g;
    const int64_t slot = is_split ? (p.max_chunks > 1 ? (int64_t)p.B * p.Hkv * p.n_sink_kt * p.max_chunks : 0) +
                                        (bg * p.n_split_kt + (xt - p.split_kt0())) * p.split_chunks + chunk
                                  : (bg * p.n_sink_kt + xt) * p.max_chunks + chunk;
    return BwdItem{b, g, xt, yt_begin, yt_start, nt, partial, slot};
}

}  // namespace loza
#endif
