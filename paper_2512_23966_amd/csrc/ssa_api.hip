// C ABI of the SSA library: argument validation, host-side schedule arithmetic, dispatch.
// Every check runs before the first HIP call, so a rejected call launches nothing.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <mutex>

#include "../../include/loza_ssa.h"
#include "ssa_kernels.h"
#include "ssa_schedule.h"

// Scratch memory of loza_ssa_decode_static: the split kernel's partial results, in the place of a
// caller's workspace. One copy per GPU, at an address of its own on each; the name below is only a
// host-side handle for hipGetSymbolAddress and is never passed to a kernel.
static __device__ __align__(256) unsigned char scratch[LOZA_DECODE_STATIC_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_ptr[kMaxDevices];      // device address of `scratch` on device d (nullptr: not asked yet)

// Device address of the scratch array on the current device (asked once per device, then kept).
int scratch_of_current_device(void **ptr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LOZA_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (scratch_ptr[dev] == nullptr) {
        void *a = nullptr;
        if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || a == nullptr) return LOZA_ERR_HIP;
        scratch_ptr[dev] = a;
    }
    *ptr = scratch_ptr[dev];
    return LOZA_OK;
}

constexpr int kComputeUnits = 256;              // MI355X
constexpr int64_t kMaxSeq = 2147483647LL - 128;  // positions are 32-bit inside the kernels
constexpr int kMaxSplits = 64;                   // key splits of a decode query, at most

inline bool aligned16(const void *ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

// window / n_sink cut to what can matter for sequences of at most S keys
inline int clamp_to(int64_t x, int64_t S) { return (int)(x < S ? x : S); }

int check_common(int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v, int64_t n_sink, int64_t window, float scale)
{
    if (B < 1 || Hq < 1 || Hkv < 1 || S < 1 || d_qk < 1 || d_v < 1) return LOZA_ERR_SHAPE;
    if (Hq % Hkv != 0) return LOZA_ERR_SHAPE;
    if (S > kMaxSeq) return LOZA_ERR_SHAPE;
    if (n_sink < 0 || window < 1) return LOZA_ERR_SHAPE;
    if (!(scale == scale) || isinf(scale)) return LOZA_ERR_SHAPE;
    return LOZA_OK;
}

// LOZA_DECODE_SPLITS (documented in the header): another split count, for tests and experiments; 0: none given
int forced_splits()
{
    const char *env = getenv("LOZA_DECODE_SPLITS");
    const long v = env ? strtol(env, nullptr, 10) : 0;
    return v >= 1 && v <= kMaxSplits ? (int)v : 0;
}

// The split count a workspace is sized for. A call uses as many or fewer (decode_plan).
int decode_splits(int B, int Hq, int Hkv, int64_t S_max, int64_t n_sink, int64_t window)
{
    const int G = Hq / Hkv;
    const int rows = loza::decode_rows_per_tile();
    const int64_t base = (int64_t)B * Hkv * ((G + rows - 1) / rows);
    // both terms are cut to S_max before they are added: either may be INT64_MAX
    int64_t live = (n_sink < S_max ? n_sink : S_max) + (window < S_max ? window : S_max);
    if (live > S_max) live = S_max;
    const int64_t tiles = (live + 63) / 64 + 2;
    int64_t n = (kComputeUnits + base - 1) / base;  // one workgroup per compute unit at least
    if (const int v = forced_splits()) n = v;
    if (n > tiles) n = tiles;
    if (n > kMaxSplits) n = kMaxSplits;
    if (n < 1) n = 1;
    return (int)n;
}

// Which of the two decode kernels takes a call, and in how many splits (at most `most`, which the
// workspace is sized for): as many as leave the launch within one round of 256 workgroups, one at least (a
// workgroup of the wide shape fills a compute unit's LDS: 43 sequences in 6 splits of the tile kernel are 258
// workgroups, two rounds, 60 us against 33 in 5). Counts that do not divide 256 leave units idle (43 sequences
// of four groups: 172 workgroups), and beyond 256 the last round may be a short one.
// Up to two groups of 16 query heads per key head the row kernel is always the faster (d = 128, four query heads
// on each of 8 key heads, 16 sequences, window 4096: 48 against 74 us; 128 sequences on one key head of 32: 108
// against 128). With more groups (absorbed MLA: four) it reads the keys once per group, from L2, where the
// tile kernel reads them once but leaves fp32 partial results of every split; it wins until the live keys
// per split outweigh that. The line is a time model of either, in hundredths of a microsecond, fitted to the
// measured times of both (MLA, row against tile kernel: window 8192, 8 sequences 40 against 50 us, 16 65 against
// 56, 64 220 against 131; 2,176 keys, 8 sequences 22 against 38, 64 62 against 58; the paper's 1,024 keys, 16
// sequences 23 against 32; without queries that the tile kernel computes again, 250 us more). Over 161 sizes
// the kernel taken is the faster one or within 7 % of it.
struct DecodePlan {
    bool rows;
    int n_splits;
};

DecodePlan decode_plan(int B, int Hq, int Hkv, int64_t S_max, int d_qk, int64_t n_sink, int64_t window)
{
    const int G = Hq / Hkv, most = decode_splits(B, Hq, Hkv, S_max, n_sink, window);
    int64_t live = (n_sink < S_max ? n_sink : S_max) + (window < S_max ? window : S_max);
    if (live > S_max) live = S_max;
    const int64_t groups = (G + 15) / 16, rows_base = (int64_t)B * Hkv * groups;
    const int64_t tile_base = (int64_t)B * Hkv * ((G + loza::decode_rows_per_tile() - 1) / loza::decode_rows_per_tile());
    auto cut = [&](int64_t base) { const int64_t n = kComputeUnits / base; return (int)(n < 1 ? 1 : n < most ? n : most); };
    int n_rows = cut(rows_base), n_tile = cut(tile_base);
    if (forced_splits()) n_rows = n_tile = most;
    if (groups <= 2) return {true, n_rows};
    const bool wide = d_qk > 128;
    const int64_t keys = (live + 63) / 64 * 64;
    auto rounds = [&](int64_t base, int n) { return ceil((double)base * n / kComputeUnits); };
    const int64_t rows_tiles = (keys / 64 + n_rows) / n_rows, tile_tiles = (keys / 32 + n_tile) / n_tile;
    const double t_rows = rounds(rows_base, n_rows) * (rows_tiles * (wide ? 145 : 70) + (wide ? 800 : 600)) + (n_rows > 1 ? 500 : 0);
    const double t_tile = rounds(tile_base, n_tile) * (tile_tiles * (wide ? 120 : 80) + (wide ? 2500 : 1800)) + 800;
    return {t_rows <= t_tile, t_rows <= t_tile ? n_rows : n_tile};
}

// The pattern as the kernels take it: sink in tokens, window in blocks of `block` tokens, both cut
// to what can matter for S keys. The token-granular entry points use block = 1.
struct Pattern {
    int n_sink, window, block;
};

inline int64_t sat_mul(int64_t a, int64_t b) { return (a != 0 && b > INT64_MAX / a) ? INT64_MAX : a * b; }

Pattern token_pattern(int64_t n_sink, int64_t window, int64_t S)
{
    return Pattern{clamp_to(n_sink, S), clamp_to(window, S), 1};
}

// block-granular: sink_blocks >= 0, local_blocks >= 1, block >= 1 (checked by the caller)
Pattern block_pattern(int64_t sink_blocks, int64_t local_blocks, int64_t block, int64_t S)
{
    const int64_t b = block < S ? block : S;  // one block already covers everything
    if (block >= S) return Pattern{sink_blocks > 0 ? (int)S : 0, 1, (int)b};
    return Pattern{clamp_to(sat_mul(sink_blocks, block), S), clamp_to(local_blocks, S / block + 1), (int)b};
}

int check_blocks(int64_t sink_blocks, int64_t local_blocks, int64_t block)
{
    return (sink_blocks < 0 || local_blocks < 1 || block < 1) ? LOZA_ERR_SHAPE : LOZA_OK;
}

// How many workgroups share the keys of a row in an extend that has scratch memory, and of which kernel (1: no sharing,
// the kernel that takes the call without scratch memory). Few
// new tokens leave most compute units idle: 2 tokens of one sequence are 8 groups of 16 rows of the absorbed-MLA
// shape, and took the same 153 us (window 8192) as 128 tokens. Splits of the few-rows kernel are merged row by row
// (2 tokens 22 us, 16 tokens 57); calls too large for that kernel split the tile kernel's keys, until its tiles
// fill the chip by themselves, and so do calls of the few-rows kernel at the wide shape where the model says so (window
// 8192: 8 sequences of 10 tokens 294 us, their tiles in 6 parts 141; 8 of 16 302 and in 4 195; 8 of 4 the rows in 2 parts
// 93, the tiles in 16 79; 1 + 7 blocks, 8 of 16 52, tiles in 4 56: rows). Those whose groups are one full round of the
// few-rows kernel are left to it, and need no scratch memory, though tiles would be faster there, too (129 to 256 groups; 16 of 4
// tokens 160, in 8 parts 138, and 17 of 4 in 7 parts 130). The host knows windows, not lengths: where caches are short, a
// split costs 3 to 24 us (200 to 400 rows: 2 tokens 12 -> 15, 8 of 16 30 -> 44, 8 of 4 15 -> 39). A split tile has two-term weights throughout (2.45 us a step, 1.45 with weights rounded
// once): which rows have a large result is known only when the parts have been added, and a tile that has one may keep
// none of its rows from once-rounded weights. 144 tokens of window 8192 391 -> 259 us, 256 tokens 397 -> 361 in two
// parts. (d = 128, 8 key heads, window 4096: 280 tokens 154 -> 71, 600 tokens 156 -> 120.) Calls of the 256-row tiles of
// width 128 have enough workgroups, and tiles twice as fast (3 sequences of 385 tokens 130 us, as three parts of the
// 128-row tiles 212). The line is a time model of both in microseconds, fitted to 260 sizes: workgroups go in
// rounds, a round costs a start and a step per tile of keys, every row has a workgroup of the merge, and every set of
// partial results of a row is written and read once; the host's part counts, since a short call waits for it (28
// tokens of 1 + 7 blocks 25.6 us, in two parts 28.5 and 5 of the host; d = 128, 4 tokens 12.2, in 16 parts 8.5 and 5:
// not split; 8 tokens 24.4 and 17.3 + 5). A split has to promise 7 %, which is what the
// model is worth. But where one round holds all unsplit tiles of the wide shape, it may cost 7 %: an unsplit tile with a large result
// is computed again behind all others, and how often that is depends on values (us unsplit where none is, where one is, and split; 72 tiles
// of 1 + 7 blocks 65, 152, 62 in 3 parts; 100 of window 2048 116, 296, 113; 128 of window 4096 209, 536, 204; but 104 of 1 + 7 blocks
// 65, 152 and 71 in two: not split). A chunk that (nearly) fills its cache is a prefill, and has its bits.
struct ExtendPlan {
    bool rows;      // few-rows kernel, else tiles
    int n_splits;
};

// least: the plan for a workspace that does not hold the other's partial results: calls are split by the kernel that takes
// them without scratch memory alone (most of those the other gives to tiles are not split then and need none), and a
// split tile counts 2.7 us a step, which is what the sizes that callers may have kept were given out by.
ExtendPlan extend_plan(int B, int Hkv, int G, int64_t q_len, int64_t S, int d_qk, const Pattern &pat, bool least = false)
{
    const bool wide = d_qk > 128;
    const int64_t rows = q_len * G, heads = (int64_t)B * Hkv, groups = (rows + 15) / 16 * heads;
    const int64_t tiles = (rows + loza::kTileRows - 1) / loza::kTileRows * heads;
    int64_t live = (int64_t)pat.n_sink + (int64_t)pat.window * pat.block;
    if (live > S) live = S;
    auto rounds = [](int64_t workgroups, int slots) { return (double)((workgroups + slots - 1) / slots); };
    const double host = 5;                                             // of a call with scratch memory: to get it, and a launch
    auto t_rows = [&](int64_t n) {
        const double steps = (double)((live / 16 + 2 + 4 * n - 1) / (4 * n)), all = (double)(rows * heads);
        return rounds(groups * n, kComputeUnits) * (wide ? 6.5 + 1.08 * steps : 3.7 + 0.55 * steps) +
               (n > 1 ? host + (wide ? 2.5 + all * (2.8e-3 + 1.17e-3 * n) : 3.2 + all * (0.4e-3 + 0.25e-3 * n)) : 0);
    };
    // (two workgroups of the narrow tile kernel share a compute unit)
    const int slots = wide ? kComputeUnits : 2 * kComputeUnits;
    auto t_tile = [&](int64_t n) {
        const double steps = (double)((live / 32 + 2 + n - 1) / n);
        const bool alone = tiles * n <= kComputeUnits;
        const double step = n > 1 ? (wide ? (least ? 2.7 : 2.45) : alone ? 1.4 : 2.0) : (wide ? 1.45 : alone ? 1.05 : 1.36);
        return rounds(tiles * n, slots) * (12 + step * steps) + (n > 1 ? host + 6 + (wide ? 0.45e-3 : 0.11e-3) * rows * heads * n : 0);
    };
    const bool few = loza::few_rows_bf16(B, Hkv, rows);
    ExtendPlan best{few, 1};
    if (S * 8 <= q_len * 9) return best;
    if (!few && !wide && loza::d128_tiles_pay(B, Hkv, G, q_len, S, pat.n_sink, pat.window, pat.block)) return best;
    double t = 0.93 * (few ? t_rows(1) : t_tile(1));
    if (!least && !few && wide && tiles <= kComputeUnits) t *= 1.07 / 0.93;
    auto offer = [&](bool by_rows, int n, double t_n) { if (t_n < t) { t = t_n; best = ExtendPlan{by_rows, n}; } };
    for (int n = 2; few && n <= kMaxSplits && groups * n <= kComputeUnits; ++n) offer(true, n, t_rows(n));
    if (best.n_splits > 1) t *= 0.93;                                  // (so has another kernel)
    const bool by_tiles = !few || (!least && wide && (groups * 2 <= kComputeUnits || groups > kComputeUnits));
    for (int n = 2; by_tiles && n <= kMaxSplits && tiles * n <= 2 * slots; ++n) offer(false, n, t_tile(n));
    return best;
}

// The reference maximum of the online softmax moves only when exceeded by more than 2^8 (fp32 has the headroom).
// Over the first 8 key tiles the tile kernel keeps it exact (its wide prefill over the first only); the few-rows
// and the width-128 kernel, which do not read exact_tiles, over their first tile or step.
void set_rescale_policy(loza::FwdParams &p)
{
    p.exact_tiles = 8;
    p.lazy_log2 = 8.0f;
}

}  // namespace

extern "C" {

const char *loza_status_str(int status)
{
    switch (status) {
    case LOZA_OK: return "LOZA_OK";
    case LOZA_ERR_NULL: return "LOZA_ERR_NULL: a required pointer is NULL";
    case LOZA_ERR_SHAPE: return "LOZA_ERR_SHAPE: sizes out of range or inconsistent";
    case LOZA_ERR_UNSUPPORTED: return "LOZA_ERR_UNSUPPORTED: no kernel for this (dtype, d_qk, d_v)";
    case LOZA_ERR_WORKSPACE: return "LOZA_ERR_WORKSPACE: workspace missing or too small";
    case LOZA_ERR_HIP: return "LOZA_ERR_HIP: a HIP call failed";
    case LOZA_ERR_ALIGN: return "LOZA_ERR_ALIGN: a base pointer is not 16-byte aligned";
    default: return "unknown loza status";
    }
}

int loza_ssa_live_ranges(int64_t i, int64_t n_sink, int64_t window,
                         int64_t *sink_end, int64_t *win_begin, int64_t *win_end)
{
    if (!sink_end || !win_begin || !win_end) return LOZA_ERR_NULL;
    if (i < 0 || i == INT64_MAX || n_sink < 0 || window < 1) return LOZA_ERR_SHAPE;  // i + 1 is returned
    const int64_t se = n_sink < i + 1 ? n_sink : i + 1;
    int64_t wb = window > i ? 0 : i - window + 1;
    if (wb < se) wb = se;  // a key in both sets is used once
    *sink_end = se;
    *win_begin = wb;
    *win_end = i + 1;
    return LOZA_OK;
}

int loza_ssa_live_ranges_blocks(int64_t i, int64_t sink_blocks, int64_t local_blocks, int64_t block,
                                int64_t *sink_end, int64_t *win_begin, int64_t *win_end)
{
    if (!sink_end || !win_begin || !win_end) return LOZA_ERR_NULL;
    if (i < 0 || i == INT64_MAX || check_blocks(sink_blocks, local_blocks, block) != LOZA_OK) return LOZA_ERR_SHAPE;
    const int64_t sink_tokens = sat_mul(sink_blocks, block);
    const int64_t se = sink_tokens < i + 1 ? sink_tokens : i + 1;
    const int64_t qb = i / block;
    int64_t wb = local_blocks > qb ? 0 : (qb - local_blocks + 1) * block;
    if (wb < se) wb = se;
    *sink_end = se;
    *win_begin = wb;
    *win_end = i + 1;
    return LOZA_OK;
}

int64_t loza_ssa_live_pairs_blocks(int64_t S, int64_t sink_blocks, int64_t local_blocks, int64_t block)
{
    if (S < 1 || S > kMaxSeq || check_blocks(sink_blocks, local_blocks, block) != LOZA_OK) return -1;
    // query block by query block: inside one block the window start is fixed and |live(i)| grows by one
    const int64_t sink_tokens = sat_mul(sink_blocks, block);
    if (block > S) block = S;  // one block already holds every position (and i0 + block cannot overflow)
    int64_t pairs = 0;
    for (int64_t i0 = 0; i0 < S; i0 += block) {
        const int64_t i1 = (i0 + block < S ? i0 + block : S) - 1;  // last query of the block
        const int64_t qb = i0 / block;
        const int64_t wb = local_blocks > qb ? 0 : (qb - local_blocks + 1) * block;
        const int64_t n = i1 - i0 + 1;
        if (wb <= sink_tokens) {
            pairs += n * (i0 + 1) + n * (n - 1) / 2;                       // everything up to the query
        } else {
            pairs += n * (sink_tokens + i0 + 1 - wb) + n * (n - 1) / 2;    // sink + [wb, i]
        }
    }
    return pairs;
}

int64_t loza_ssa_live_pairs(int64_t S, int64_t n_sink, int64_t window)
{
    if (S < 1 || S > kMaxSeq || n_sink < 0 || window < 1) return -1;
    // |live(i)| = min(i + 1, T), T = n_sink + window (saturating)
    const int64_t T = (window >= S || n_sink >= S || n_sink + window >= S) ? S : n_sink + window;
    return T * (T + 1) / 2 + (S - T) * T;
}

// Paged cache description (block_table == nullptr: contiguous cache of S_max rows per sequence).
struct Paging {
    const int32_t *block_table;
    int64_t num_pages;
    int page_size, max_pages;
};

// Checks a paging description and gives log2(page_size) and the capacity per sequence in rows.
static int check_paging(const Paging &pg, int *page_shift, int64_t *capacity)
{
    if (!pg.block_table) return LOZA_ERR_NULL;
    // pages hold a power-of-two number of rows, at least 32: what a kernel copies at a time (16 or 32 rows; the
    // stages of 64 keys in ssa_d128.hip have a table entry for each half) lies in one page
    if (pg.page_size < 32 || (pg.page_size & (pg.page_size - 1)) != 0) return LOZA_ERR_SHAPE;
    if (pg.num_pages < 1 || pg.num_pages > 2147483647LL || pg.max_pages < 1) return LOZA_ERR_SHAPE;
    if ((int64_t)pg.max_pages * pg.page_size > kMaxSeq) return LOZA_ERR_SHAPE;
    if (reinterpret_cast<uintptr_t>(pg.block_table) & 3u) return LOZA_ERR_ALIGN;
    int s = 0;
    while ((1 << s) < pg.page_size) ++s;
    *page_shift = s;
    *capacity = (int64_t)pg.max_pages * pg.page_size;
    return LOZA_OK;
}

// Partial results of the rows of a call whose keys n workgroups share: fp32 results, then maximum and sums.
static size_t split_bytes(int B, int Hq, int64_t q_len, int d_v, int n)
{
    return (size_t)B * Hq * q_len * n * ((size_t)d_v + 4) * sizeof(float);
}

static int prefill_bf16(const void *q, const void *k, const void *v, void *out, float *lse,
                        int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                        int64_t sink, int64_t local, int64_t block, bool blocks, float scale, void *stream,
                        float *out_f32 = nullptr, bool validate_only = false,
                        const int32_t *seqlens = nullptr, int64_t q_len = 0, const Paging *paging = nullptr,
                        bool scratch = false, void *workspace = nullptr, size_t workspace_bytes = 0)
{
    // seqlens != nullptr: "extend" form, q_len queries per sequence against a cache of S rows
    // (with a paging description: of max_pages * page_size rows behind a block table); scratch: the caller offers
    // `workspace`, and the keys of a row may be shared by several workgroups
    const bool extend = seqlens != nullptr;
    if (!q || !k || !v || (!out && !out_f32) || !lse) return LOZA_ERR_NULL;
    int page_shift = 0;
    if (paging) {
        if (!extend) return LOZA_ERR_SHAPE;
        if (int rc = check_paging(*paging, &page_shift, &S)) return rc;
    }
    if (extend && (q_len < 1 || q_len > S || (reinterpret_cast<uintptr_t>(seqlens) & 3u))) return q_len < 1 || q_len > S ? LOZA_ERR_SHAPE : LOZA_ERR_ALIGN;
    if (int rc = check_common(B, Hq, Hkv, S, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    if (!(scale > 0.f)) return LOZA_ERR_SHAPE;  // the row maximum is taken before the scaling
    const bool alias = (v == k);
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (!loza::bf16_shape_supported(d_qk, d_v, alias)) return LOZA_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse)) return LOZA_ERR_ALIGN;
    const int G = Hq / Hkv;
    const int rows = loza::prefill_rows_per_tile();
    const int64_t row_tiles = ((extend ? q_len : S) * G + rows - 1) / rows;
    if (row_tiles * Hkv * B > 2147483647LL) return LOZA_ERR_SHAPE;
    if (validate_only) return LOZA_OK;

    loza::FwdParams p{};
    p.q = (const uint16_t *)q; p.k = (const uint16_t *)k; p.v = (const uint16_t *)v;
    p.out = (uint16_t *)out; p.out_f32 = out_f32; p.lse = lse;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.G = G; p.S = S;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S) : token_pattern(sink, local, S);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale_log2 = scale * 1.44269504088896340736f;
    p.row_tiles = (int)row_tiles; p.n_splits = 1;
    set_rescale_policy(p);
    bool few_rows = loza::few_rows_bf16(B, Hkv, (extend ? q_len : S) * G);
    if (extend) {
        if (scratch) {
            auto held = [&](int n) { return n == 1 || (workspace && workspace_bytes >= split_bytes(B, Hq, q_len, d_v, n)); };
            ExtendPlan plan = extend_plan(B, Hkv, G, q_len, S, d_qk, pat);
            if (!held(plan.n_splits)) plan = extend_plan(B, Hkv, G, q_len, S, d_qk, pat, true);
            if (!held(plan.n_splits)) return LOZA_ERR_WORKSPACE;
            few_rows = plan.rows;
            p.n_splits = plan.n_splits;
            if (p.n_splits > 1) {
                if (!aligned16(workspace)) return LOZA_ERR_ALIGN;
                p.part_o = (float *)workspace;
                p.part_ml = (float *)workspace + (size_t)B * Hq * q_len * p.n_splits * d_v;
            }
        }
        p.seqlens = seqlens; p.q_len = (int)q_len;
        if (paging) {
            p.block_table = paging->block_table;
            p.page_shift = page_shift; p.max_pages = paging->max_pages; p.num_pages = (int)paging->num_pages;
        }
        if (few_rows) return loza::launch_rows_bf16(p, d_qk, d_v, alias, false, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
        return loza::launch_extend_bf16(p, d_qk, d_v, alias, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
    }
    if (few_rows) return loza::launch_rows_bf16(p, d_qk, d_v, alias, false, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
    return loza::launch_prefill_bf16(p, d_qk, d_v, alias, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_forward_kernel(int B, int Hq, int Hkv, int64_t n_queries, int64_t S, int d_qk,
                            int64_t sink_blocks, int64_t local_blocks, int64_t block)
{
    if (int rc = check_common(B, Hq, Hkv, S, d_qk, 1, sink_blocks, local_blocks, 1.0f)) return rc;
    if (int rc = check_blocks(sink_blocks, local_blocks, block)) return rc;
    if (n_queries < 1 || n_queries > S) return LOZA_ERR_SHAPE;
    if (!loza::bf16_width_supported(d_qk)) return LOZA_ERR_UNSUPPORTED;
    const int G = Hq / Hkv;
    if (loza::few_rows_bf16(B, Hkv, n_queries * G)) return LOZA_KERNEL_ROWS;
    const Pattern pat = block_pattern(sink_blocks, local_blocks, block, S);
    return d_qk == 128 && loza::d128_tiles_pay(B, Hkv, G, n_queries, S, pat.n_sink, pat.window, pat.block) ? LOZA_KERNEL_D128 : LOZA_KERNEL_TILES;
}

int loza_ssa_extend(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens, void *out, float *lse,
                    int B, int Hq, int Hkv, int64_t S_max, int q_len, int d_qk, int d_v,
                    int64_t n_sink, int64_t window, float scale, void *stream)
{
    if (!seqlens) return LOZA_ERR_NULL;
    return prefill_bf16(q, kcache, vcache, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, n_sink, window, 1, false, scale, stream,
                        nullptr, false, seqlens, q_len);
}

int loza_ssa_extend_paged(const void *q, const void *k_pages, const void *v_pages, const int32_t *block_table,
                          const int32_t *seqlens, void *out, float *lse, int B, int Hq, int Hkv,
                          int64_t num_pages, int page_size, int max_pages_per_seq, int q_len, int d_qk, int d_v,
                          int64_t n_sink, int64_t window, float scale, void *stream)
{
    if (!seqlens) return LOZA_ERR_NULL;
    const Paging pg{block_table, num_pages, page_size, max_pages_per_seq};
    return prefill_bf16(q, k_pages, v_pages, out, lse, B, Hq, Hkv, 1, d_qk, d_v, n_sink, window, 1, false, scale, stream,
                        nullptr, false, seqlens, q_len, &pg);
}

int loza_ssa_extend_paged_blocks(const void *q, const void *k_pages, const void *v_pages, const int32_t *block_table,
                                 const int32_t *seqlens, void *out, float *lse, int B, int Hq, int Hkv,
                                 int64_t num_pages, int page_size, int max_pages_per_seq, int q_len, int d_qk, int d_v,
                                 int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    if (!seqlens) return LOZA_ERR_NULL;
    const Paging pg{block_table, num_pages, page_size, max_pages_per_seq};
    return prefill_bf16(q, k_pages, v_pages, out, lse, B, Hq, Hkv, 1, d_qk, d_v, sink_blocks, local_blocks, block, true,
                        scale, stream, nullptr, false, seqlens, q_len, &pg);
}

int loza_ssa_extend_blocks(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens, void *out,
                           float *lse, int B, int Hq, int Hkv, int64_t S_max, int q_len, int d_qk, int d_v,
                           int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    if (!seqlens) return LOZA_ERR_NULL;
    return prefill_bf16(q, kcache, vcache, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, sink_blocks, local_blocks, block, true,
                        scale, stream, nullptr, false, seqlens, q_len);
}

int loza_ssa_extend_with_workspace(const void *q, const void *k, const void *v, const int32_t *block_table, const int32_t *seqlens,
                                   void *out, float *lse, int B, int Hq, int Hkv, int64_t S_max, int64_t num_pages,
                                   int page_size, int max_pages_per_seq, int q_len, int d_qk, int d_v, int64_t sink_blocks,
                                   int64_t local_blocks, int64_t block, float scale, void *workspace, size_t workspace_bytes,
                                   void *stream)
{
    if (!seqlens) return LOZA_ERR_NULL;
    const Paging pg{block_table, num_pages, page_size, max_pages_per_seq};
    return prefill_bf16(q, k, v, out, lse, B, Hq, Hkv, block_table ? 1 : S_max, d_qk, d_v, sink_blocks, local_blocks, block, true,
                        scale, stream, nullptr, false, seqlens, q_len, block_table ? &pg : nullptr, true, workspace, workspace_bytes);
}

size_t loza_ssa_extend_workspace_bytes(int B, int Hq, int Hkv, int64_t S_max, int q_len, int d_qk, int d_v,
                                       int64_t sink_blocks, int64_t local_blocks, int64_t block)
{
    if (check_common(B, Hq, Hkv, S_max, d_qk, d_v, sink_blocks, local_blocks, 1.0f) != LOZA_OK) return 0;
    if (check_blocks(sink_blocks, local_blocks, block) != LOZA_OK || q_len < 1 || q_len > S_max) return 0;
    if (!loza::bf16_width_supported(d_qk)) return 0;
    const int n = extend_plan(B, Hkv, Hq / Hkv, q_len, S_max, d_qk, block_pattern(sink_blocks, local_blocks, block, S_max)).n_splits;
    return n > 1 ? split_bytes(B, Hq, q_len, d_v, n) : 0;
}

int loza_ssa_prefill(const void *q, const void *k, const void *v, void *out, float *lse,
                     int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                     int64_t n_sink, int64_t window, float scale, void *stream)
{
    return prefill_bf16(q, k, v, out, lse, B, Hq, Hkv, S, d_qk, d_v, n_sink, window, 1, false, scale, stream);
}

int loza_ssa_prefill_blocks(const void *q, const void *k, const void *v, void *out, float *lse,
                            int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                            int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    return prefill_bf16(q, k, v, out, lse, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true, scale, stream);
}

static int prefill_f32(const float *q, const float *k, const float *v, float *out, float *lse,
                       int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                       int64_t sink, int64_t local, int64_t block, bool blocks, float scale, void *stream)
{
    if (!q || !k || !v || !out || !lse) return LOZA_ERR_NULL;
    if (int rc = check_common(B, Hq, Hkv, S, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    const bool alias = (v == k);
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (d_qk > 256 || d_v > 256) return LOZA_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse)) return LOZA_ERR_ALIGN;
    if (((int64_t)B * S * Hq + 3) / 4 > 2147483647LL) return LOZA_ERR_SHAPE;

    loza::F32Params p{};
    p.q = q; p.k = k; p.v = v; p.out = out; p.lse = lse;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.S = S; p.d_qk = d_qk; p.d_v = d_v;
    p.k_row = d_qk; p.v_row = alias ? d_qk : d_v;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S) : token_pattern(sink, local, S);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale = scale;
    return loza::launch_prefill_f32(p, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

static int decode_f32(const float *q, const float *kcache, const float *vcache, const int32_t *seqlens, float *out, float *lse,
                      int B, int Hq, int Hkv, int64_t S_max, int d_qk, int d_v,
                      int64_t sink, int64_t local, int64_t block, bool blocks, float scale, void *stream)
{
    if (!q || !kcache || !vcache || !seqlens || !out || !lse) return LOZA_ERR_NULL;
    if (int rc = check_common(B, Hq, Hkv, S_max, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    const bool alias = (vcache == kcache);
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (d_qk > 256 || d_v > 256) return LOZA_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(kcache) || !aligned16(vcache) || !aligned16(out) ||
        (reinterpret_cast<uintptr_t>(seqlens) & 3u) || (reinterpret_cast<uintptr_t>(lse) & 3u))
        return LOZA_ERR_ALIGN;
    if (((int64_t)B * Hq + 3) / 4 > 2147483647LL) return LOZA_ERR_SHAPE;

    loza::F32Params p{};
    p.q = q; p.k = kcache; p.v = vcache; p.out = out; p.lse = lse; p.seqlens = seqlens;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.S = S_max; p.d_qk = d_qk; p.d_v = d_v;
    p.k_row = d_qk; p.v_row = alias ? d_qk : d_v;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S_max) : token_pattern(sink, local, S_max);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale = scale;
    return loza::launch_prefill_f32(p, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_decode_f32(const float *q, const float *kcache, const float *vcache, const int32_t *seqlens, float *out, float *lse,
                        int B, int Hq, int Hkv, int64_t S_max, int d_qk, int d_v,
                        int64_t n_sink, int64_t window, float scale, void *stream)
{
    return decode_f32(q, kcache, vcache, seqlens, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, n_sink, window, 1, false, scale, stream);
}

int loza_ssa_decode_blocks_f32(const float *q, const float *kcache, const float *vcache, const int32_t *seqlens, float *out,
                               float *lse, int B, int Hq, int Hkv, int64_t S_max, int d_qk, int d_v,
                               int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    return decode_f32(q, kcache, vcache, seqlens, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, sink_blocks, local_blocks, block, true,
                      scale, stream);
}

size_t loza_ssa_calibration_workspace_bytes(int B, int Hq, int64_t S, int d_v)
{
    if (B < 1 || Hq < 1 || S < 1 || d_v < 1 || S > kMaxSeq) return 0;
    return (size_t)2 * B * S * Hq * d_v * sizeof(float);
}

int loza_ssa_prefill_calibration_blocks(const void *q, const void *k, const void *v,
                                        void *out, void *out_full, void *out_sparse, float *lse_full, float *lse_sparse,
                                        int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                        int64_t sink_blocks, int64_t local_blocks, int64_t block,
                                        float alpha, float scale, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!out || !lse_full || !lse_sparse) return LOZA_ERR_NULL;
    if (!(alpha >= 0.f && alpha <= 1.f)) return LOZA_ERR_SHAPE;
    const size_t need = loza_ssa_calibration_workspace_bytes(B, Hq, S, d_v);
    if (need == 0) return LOZA_ERR_SHAPE;
    if (!workspace || workspace_bytes < need) return LOZA_ERR_WORKSPACE;
    if (!aligned16(out) || !aligned16(workspace) || (out_full && !aligned16(out_full)) || (out_sparse && !aligned16(out_sparse)))
        return LOZA_ERR_ALIGN;
    float *o_full = (float *)workspace, *o_sparse = o_full + need / (2 * sizeof(float));
    // every argument of both passes is checked before the first launch
    if (int rc = prefill_bf16(q, k, v, nullptr, lse_full, B, Hq, Hkv, S, d_qk, d_v, 0, 1, INT64_MAX, true, scale, stream, o_full, true))
        return rc;
    if (int rc = prefill_bf16(q, k, v, nullptr, lse_sparse, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true,
                              scale, stream, o_sparse, true))
        return rc;
    // O: every causal key (one block that holds everything); O': the sparse pattern
    if (int rc = prefill_bf16(q, k, v, nullptr, lse_full, B, Hq, Hkv, S, d_qk, d_v, 0, 1, INT64_MAX, true, scale, stream, o_full))
        return rc;
    if (int rc = prefill_bf16(q, k, v, nullptr, lse_sparse, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true,
                              scale, stream, o_sparse))
        return rc;
    const int64_t n = (int64_t)B * S * Hq * d_v;  // a multiple of 8: d_v is
    return loza::launch_blend_bf16(o_full, o_sparse, alpha, (uint16_t *)out, (uint16_t *)out_full, (uint16_t *)out_sparse, n,
                                   (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

size_t loza_ssa_calibration_alpha_grad_workspace_bytes(int64_t n)
{
    if (n < 8 || n % 8 != 0) return 0;
    return (size_t)loza::alpha_grad_blocks(n) * sizeof(double);
}

int loza_ssa_calibration_alpha_grad(const void *dout, const void *out_full, const void *out_sparse, float *dalpha, int64_t n,
                                    void *workspace, size_t workspace_bytes, void *stream)
{
    if (!dout || !out_full || !out_sparse || !dalpha) return LOZA_ERR_NULL;
    const size_t need = loza_ssa_calibration_alpha_grad_workspace_bytes(n);
    if (need == 0) return LOZA_ERR_SHAPE;
    if (!workspace || workspace_bytes < need) return LOZA_ERR_WORKSPACE;
    if (!aligned16(dout) || !aligned16(out_full) || !aligned16(out_sparse) || !aligned16(workspace) ||
        (reinterpret_cast<uintptr_t>(dalpha) & 3u))
        return LOZA_ERR_ALIGN;
    return loza::launch_alpha_grad_bf16((const uint16_t *)dout, (const uint16_t *)out_full, (const uint16_t *)out_sparse, dalpha, n,
                                        (double *)workspace, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_prefill_f32(const float *q, const float *k, const float *v, float *out, float *lse,
                         int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                         int64_t n_sink, int64_t window, float scale, void *stream)
{
    return prefill_f32(q, k, v, out, lse, B, Hq, Hkv, S, d_qk, d_v, n_sink, window, 1, false, scale, stream);
}

int loza_ssa_prefill_blocks_f32(const float *q, const float *k, const float *v, float *out, float *lse,
                                int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    return prefill_f32(q, k, v, out, lse, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true, scale, stream);
}

// ---- backward ---------------------------------------------------------------------------------------

// Host-side schedule of the key-stationary backward kernel: how many key tiles hold sink keys (their
// rows run in chunks as workgroups of their own), how long a chunk is, how many the first tile has.
static void backward_plan(loza::BwdParams &p)
{
    const int64_t n_kt = (p.S + 63) / 64;
    const int64_t sink_kt = ((int64_t)p.n_sink + 63) / 64;
    p.n_sink_kt = (int)(sink_kt < n_kt ? sink_kt : n_kt);
    // a chunk is as long as the row range of a key tile without sink keys (64 keys + the window's reach)
    const int64_t reach = (int64_t)p.window * p.block + 64 + p.block;
    int64_t ct = ((reach < p.S ? reach : p.S) * p.G + 31) / 32 + 1;
    if (ct < 64) ct = 64;
    p.chunk_tiles = (int)ct;
    int lo, hi;
    loza::bwd_key_tile_rows(p, 0, lo, hi);
    p.max_chunks = p.n_sink_kt > 0 ? (int)((hi - lo + 1 + ct - 1) / ct) : 1;
}

// Time of the key-stationary kernel's launch by the model of ssa_schedule.h, in row tiles of work: a compute unit
// holds one workgroup of the wide shape and two of width 128 (each of two then has 0.8 of its speed alone). Of the
// wide shape a row tile of a chunk that is split for balance counts 1.2: it writes fp32 partial sums that are
// read back, and fewer workgroups share the rows it streams. With these constants the model sides with the
// measured times of 130 plans, whole against split, but for one that it takes whole and loses 2 %.
static float backward_time(const loza::BwdParams &p, bool wide)
{
    const int64_t n_kt = (p.S + 63) / 64, BH = (int64_t)p.B * p.Hkv, kt0 = p.split_kt0();
    const int64_t whole = kt0 * p.max_chunks + (n_kt - kt0 - p.n_split_kt), split = (int64_t)p.n_split_kt * p.split_chunks;
    float work[9216];                                                 // of one (sequence, key head), 0: an empty chunk
    if (whole + split > 9216) return INFINITY;                        // (backward_balance asks for fewer)
    for (int64_t i = 0; i < whole + split; ++i) {
        int64_t kt, chunk = 0, ct = 0;
        if (i >= whole) { kt = kt0 + (i - whole) / p.split_chunks; chunk = (i - whole) % p.split_chunks; }
        else if (i < kt0 * p.max_chunks) { kt = i / p.max_chunks; chunk = i % p.max_chunks; ct = p.chunk_tiles; }
        else kt = i - kt0 * p.max_chunks + kt0 + p.n_split_kt;
        int lo, hi;
        loza::bwd_key_tile_rows(p, (int)kt, lo, hi);
        int64_t len = hi - lo + 1;
        if (i >= whole) ct = (len + p.split_chunks - 1) / p.split_chunks;
        if (ct > 0) len = len - chunk * ct < ct ? len - chunk * ct : ct;
        work[i] = len <= 0 ? 0.f : (float)len * (i >= whole && wide ? 1.2f : 1.f) + 16.f;
    }
    float longest = 0.f;
    for (int xcd = 0; xcd < 8; ++xcd) {
        int64_t id = xcd;
        const float t = loza::xcd_time(wide ? 1 : 2, 0.8f, [&]() {
            float w = 0.f;
            for (; id < (whole + split) * BH && w == 0.f; id += 8) {
                // (the kernel's own way from a workgroup's number to its work)
                const int64_t n = id < whole * BH ? whole : split, x = id < whole * BH ? id : id - whole * BH, eighth = n * BH / 8;
                const int64_t item = (x < eighth * 8 ? x % 8 * eighth + x / 8 : x) % n;
                w = work[id < whole * BH ? item : whole + item];
            }
            return w;
        });
        if (t > longest) longest = t;
    }
    return longest;
}

// The key-stationary kernel's work items are key tiles and chunks of sink tiles: what is left over after the
// last full round of 256 is cut into chunks that fill the chip where that ends sooner by the model above (16,384 tokens of 1 + 7 blocks of 128, absorbed MLA: 286 items ran two
// rounds, 9.0 ms; 256 whole ones and 30 in 8 chunks each: 6.0. 16,384 tokens of 128 + 8192: 258 items, of which
// the last are short; in chunks 57 ms forward and backward, whole 53). The chunks leave fp32 partial sums in
// `dq`, which is free until the row-stationary kernel writes it (the workspace is sized without them); where
// that does not hold them, the plan stays as it is.
static void backward_balance(loza::BwdParams &p, int d_qk, int d_v, bool alias)
{
    const int64_t n_kt = (p.S + 63) / 64, BH = (int64_t)p.B * p.Hkv, cus = kComputeUnits;
    const int64_t cols = alias ? d_qk : d_qk + d_v, room = (int64_t)p.B * p.S * p.Hq * d_qk * 2 / (64 * cols * 4);
    const int64_t kt0 = p.split_kt0(), total = (kt0 * p.max_chunks + n_kt - kt0) * BH, rest = total % cus;
    if (total > 10 * cus) return;                                     // little to gain in the last of many rounds
    int lo, hi;
    loza::bwd_key_tile_rows(p, (int)(kt0 < n_kt ? kt0 : n_kt - 1), lo, hi);
    const int64_t len = hi - lo + 1;                                  // row tiles of the first tile to be split
    int64_t n_split = (rest + BH - 1) / BH;
    if (n_split > n_kt - kt0) n_split = n_kt - kt0;
    if (n_split < 1) return;
    // how many chunks: last rounds in units of a whole item, each chunk a hundredth more, all items alike
    int64_t best_k = 1, best = INT64_MAX;
    for (int64_t k = 1; k <= 16 && len / k >= 32; ++k) {
        const int64_t t = ((n_split * BH * k + cus - 1) / cus) * 1000 / k + 10 * k;
        if (t < best) { best = t; best_k = k; }
    }
    if (best_k == 1) return;
    loza::BwdParams q = p;
    q.n_split_kt = (int)n_split;
    q.split_chunks = (int)best_k;
    if (total < cus && q.max_chunks > 1) {                            // no full round: the sink tiles' chunks too
        q.chunk_tiles = (int)((p.chunk_tiles + best_k - 1) / best_k);
        loza::bwd_key_tile_rows(p, 0, lo, hi);
        q.max_chunks = (hi - lo + q.chunk_tiles) / q.chunk_tiles;
    }
    const int64_t slots = BH * ((q.max_chunks > 1 ? (int64_t)q.n_sink_kt * q.max_chunks : 0) + n_split * best_k);
    if (slots > room || backward_time(q, d_qk > 128) >= backward_time(p, d_qk > 128)) return;
    q.part = (float *)p.dq;
    p = q;
}

// Chunks and work items of the passes of ssa_bwd_wide.hip; false where the kernels of ssa_bwd.hip serve: those keep no
// weights, and start on 64 rows or keys instead of 128, so they win where a row sees 128 keys or fewer and the rounds
// of workgroups are many (us, those against the passes; 64 heads: 3,000 tokens of window 128 530 against 553, of 16 373
// against 488; 32 sequences of 128 tokens 514 against 548, of 64 sequences of 64 442 against 542; 8 of 128 175 against
// 161, 16 of 200 525 against 467; 4,000 tokens of 16 + 256 1264 against 958, 1 + 7 blocks of 128 at 16,384 9700 against
// 6850, 128 + 8192 at 12,000 39200 against 25100).
// They win, too, where a key head has few query heads, since then a group of 128 keys has few (query, key) pairs to share its
// 295 KB of partial sums: the line is 2,304 live keys of a row (the mean over the sequence) times heads a group. (One
// sequence, heads a group, tokens, pattern: 2, 11,988, 200 109 against 134; 2, 64,000, 128 + 2048 2174 against 1860; 4, 8,653, 200 x 3 sequences
// 375 against 440; 4, 8,000, 1 + 7 blocks 380 against 281; 8, 12,201, 200 x 8 2425 against 2746, 256 2725 against 2885; 8, 8,000, 1 + 7 blocks
// 731 against 486; 16 x 500 tokens of 8 heads 280 against 290; 16, 8,000, 200 tokens and more: always the passes.)
// But up to 4,096 keys in all their tiles of 64 leave most of the chip idle, and up to 8,192 where the tiles of sink keys,
// which every row sees, are the longest (4, 2,000, 1 + 7 blocks 314 against 180; 2, 2,428, 200 76 against 78; 4, 4,330, 16 + 320 221 against
// 117; with 2 heads a group 6,500 of 1 + 7 blocks 200 against 234, so not there). Nor do many key heads of very few query heads pay: four times
// their number may not exceed the square of the heads a group (1,000 tokens of 1 + 7 blocks, sequences x query heads a
// group: 1 x 1 121 against 159, 16 x 1 134 against 238, 4 x 2 182 against 185, 16 x 2 244 against 287, 4 x 4 297 against 199,
// 16 x 4 438 against 480, 64 x 8 2816 against 3229, 64 x 16 6065 against 5797). Over 1,250 shapes near these lines the passes
// are the slower ones by more than 3 % at 17 that take them, 10 % at most.
static bool backward_wide_plan(const loza::BwdParams &p, int d_qk, int d_v, bool alias, loza::WidePlan &w)
{
    if (d_qk != 576 || d_v != 512 || !alias) return false;
    const int64_t R = p.S * p.G, tiles = (R + 127) / 128, groups = (p.S + 127) / 128, BH = (int64_t)p.B * p.Hkv;
    if (groups > 32768) return false;                                // (the ring's division is exact up to there)
    const int64_t sinks = (p.n_sink + 127) / 128, reach = (int64_t)p.window * p.block;
    if (tiles * BH > 2 * kComputeUnits && (p.S <= 128 || p.n_sink + reach <= 128)) return false;
    if (4 * BH > (int64_t)p.G * p.G) return false;
    const int64_t live = p.n_sink + reach < p.S ? p.n_sink + reach : p.S;
    if (p.G * live * (2 * p.S - live) < 2304 * 2 * p.S && BH * p.S > (p.n_sink > 0 && p.G > 2 ? 8192 : 4096)) return false;
    const int64_t span = 127 / p.G + 2;                              // positions of 128 rows, at most
    const int64_t ring = (reach + span - 1 + 126) / 128 + 1;
    loza::WideChunk &c = w.chunk;
    c = loza::WideChunk{};
    c.sink_groups = (int)(sinks < groups ? sinks : groups);
    c.win_groups = (int)(ring < 2 ? 2 : ring < groups ? ring : groups < 2 ? 2 : groups);
    c.win_magic = (uint32_t)(((1ULL << 32) + c.win_groups - 1) / c.win_groups);
    c.slots = c.sink_groups + c.win_groups;
    // The weights of a chunk of rows take 2 GiB of scratch memory at most (or what 256 row tiles, a round, take: up to
    // 4): with 1, 16,384 tokens of 1 + 7 blocks of 128 take 7.4 ms instead of 6.9, with 4 or 8 7.0 and 6.8.
    const int64_t tile_bytes = (int64_t)c.slots * 65536, cap = 2LL << 30;
    w.row_tiles = (int)tiles;
    if (tiles * tile_bytes <= cap) {
        // (with the partial sums, which outweigh the weights where a key head has few query heads)
        const int64_t n = cap / (tiles * tile_bytes + groups * 128 * d_qk * (int64_t)sizeof(float));
        const int64_t chunks = n < 1 ? BH : (BH + n - 1) / n;         // (of equal size)
        w.chunk_bgs = (int)((BH + chunks - 1) / chunks);
        w.chunk_tiles = (int)tiles;
    } else {
        const int64_t n = cap / tile_bytes / 256 * 256;
        if (n < 256 && 256 * tile_bytes > 2 * cap) return false;
        w.chunk_bgs = 1;
        w.chunk_tiles = (int)(n < 256 ? 256 : n);
        if (w.chunk_tiles > tiles) w.chunk_tiles = (int)tiles;
    }
    // Segments: rounds of 256 work items, each as long as a segment and 24 row blocks more (start, end, partial sums)
    auto seen = [&](int64_t t) {                                      // key groups that t row tiles see, at most
        const int64_t n = c.sink_groups + (reach + (t * 128 - 1) / p.G + 1 + 126) / 128 + 1;
        return n < groups ? n : groups;
    };
    int64_t best = INT64_MAX;
    for (int64_t n = 1; n <= 256 && n <= w.chunk_tiles; ++n) {
        const int64_t seg = (w.chunk_tiles + n - 1) / n, items = n * w.chunk_bgs * seen(seg);
        if (n > 1 && items > 1536) break;
        const int64_t t = (items + kComputeUnits - 1) / kComputeUnits * (4 * seg + 24);
        if (t < best) { best = t; c.seg_tiles = (int)seg; }
    }
    c.n_seg = (w.chunk_tiles + c.seg_tiles - 1) / c.seg_tiles;
    c.max_groups = (int)seen(c.seg_tiles);
    w.scratch_bytes = (size_t)(w.chunk_tiles * tile_bytes) * w.chunk_bgs;
    w.part_bytes = (size_t)w.chunk_bgs * c.n_seg * c.max_groups * 128 * d_qk * sizeof(float);
    // (Places as in a row block: the groups that rows on both sides of a chunk's end see are no more than one block's. Indexed
    // by group, as it is where groups are few, it was 2.25 GiB of 4.77 at a million tokens, 64 heads, 1 + 7 blocks of 128; now 5 MB.)
    w.acc_places = w.chunk_tiles == tiles ? 0 : 2 * c.slots < groups ? 2 * c.slots : (int)groups;
    w.acc_bytes = (size_t)w.acc_places * 128 * d_qk * sizeof(float);
    return true;
}

static int backward_fill(loza::BwdParams &p, int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                         int64_t sink, int64_t local, int64_t block, bool blocks, float scale, bool alias)
{
    if (int rc = check_common(B, Hq, Hkv, S, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    if (!(scale > 0.f)) return LOZA_ERR_SHAPE;
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (!loza::bf16_shape_supported(d_qk, d_v, alias)) return LOZA_ERR_UNSUPPORTED;
    if (!loza::bwd_group_supported(Hq / Hkv)) return LOZA_ERR_UNSUPPORTED;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.G = Hq / Hkv; p.S = S;
    if (S * p.G > 2147483647LL - 64) return LOZA_ERR_SHAPE;
    p.r_pad = (S * p.G + 31) / 32 * 32;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S) : token_pattern(sink, local, S);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale = scale;
    p.scale_log2 = scale * 1.44269504088896340736f;
    backward_plan(p);
    const int64_t n_kt = (S + 63) / 64;
    const int64_t items = (int64_t)p.n_sink_kt * p.max_chunks + (n_kt - p.n_sink_kt);
    if (items * Hkv * B > 2147483647LL || ((S * p.G + 63) / 64) * Hkv * B > 2147483647LL ||
        ((int64_t)B * S * Hq + 3) / 4 > 2147483647LL)
        return LOZA_ERR_SHAPE;
    return LOZA_OK;
}

// With `wide`: what the passes of ssa_bwd_wide.hip take, else the least that a call runs with.
static size_t backward_bytes(const loza::BwdParams &p, int d_qk, int d_v, bool alias, const loza::WidePlan *wide, size_t *part_offset)
{
    size_t stat = (size_t)p.B * p.Hkv * (size_t)p.r_pad * sizeof(float2);
    stat = (stat + 255) / 256 * 256;
    if (part_offset) *part_offset = stat;
    const size_t cols = alias ? (size_t)d_qk : (size_t)d_qk + d_v;
    const size_t part = p.max_chunks > 1 ? (size_t)p.B * p.Hkv * p.n_sink_kt * p.max_chunks * 64 * cols * sizeof(float) : 0;
    return stat + (wide && wide->bytes() > part ? wide->bytes() : part);
}

static size_t backward_workspace(int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                 int64_t sink, int64_t local, int64_t block, bool blocks, int alias)
{
    loza::BwdParams p{};
    if (backward_fill(p, B, Hq, Hkv, S, d_qk, d_v, sink, local, block, blocks, 1.0f, alias != 0) != LOZA_OK) return 0;
    loza::WidePlan w;
    return backward_bytes(p, d_qk, d_v, alias != 0, backward_wide_plan(p, d_qk, d_v, alias != 0, w) ? &w : nullptr, nullptr);
}

static int backward_bf16(const void *q, const void *k, const void *v, const void *out, const float *lse,
                         const void *dout, void *dq, void *dk, void *dv,
                         int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                         int64_t sink, int64_t local, int64_t block, bool blocks, float scale,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    if (!q || !k || !v || !out || !lse || !dout || !dq || !dk) return LOZA_ERR_NULL;
    const bool alias = (v == k);
    if (!alias && !dv) return LOZA_ERR_NULL;
    loza::BwdParams p{};
    if (int rc = backward_fill(p, B, Hq, Hkv, S, d_qk, d_v, sink, local, block, blocks, scale, alias)) return rc;
    size_t part_offset = 0;
    const size_t need = backward_bytes(p, d_qk, d_v, alias, nullptr, &part_offset);
    if (!workspace || workspace_bytes < need) return LOZA_ERR_WORKSPACE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(dout) || !aligned16(dq) ||
        !aligned16(dk) || (!alias && !aligned16(dv)) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(lse) & 3u))
        return LOZA_ERR_ALIGN;
    p.q = (const uint16_t *)q; p.k = (const uint16_t *)k; p.v = (const uint16_t *)v;
    p.out = (const uint16_t *)out; p.dout = (const uint16_t *)dout; p.lse = lse;
    p.dq = (uint16_t *)dq; p.dk = (uint16_t *)dk; p.dv = alias ? nullptr : (uint16_t *)dv;
    p.rowstat = (float2 *)workspace;
    p.part = (float *)((char *)workspace + part_offset);
    loza::WidePlan w;
    const bool wide = backward_wide_plan(p, d_qk, d_v, alias, w) && workspace_bytes >= backward_bytes(p, d_qk, d_v, alias, &w, nullptr);
    if (wide) {
        w.chunk.scratch = (char *)workspace + part_offset;
        w.chunk.part = (float *)(w.chunk.scratch + w.scratch_bytes);
        w.chunk.acc_in = (float *)((char *)w.chunk.part + w.part_bytes);
        w.chunk.acc_out = (float *)((char *)w.chunk.acc_in + (w.acc_places == 2 * w.chunk.slots ? w.acc_bytes / 2 : 0));
    } else {
        backward_balance(p, d_qk, d_v, alias);
    }
    return loza::launch_backward_bf16(p, d_qk, d_v, alias, wide ? &w : nullptr, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_backward_split(int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v, int64_t sink_blocks,
                            int64_t local_blocks, int64_t block, int v_aliases_k, int *n_chunks, int64_t *n_whole)
{
    loza::BwdParams p{};
    if (int rc = backward_fill(p, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true, 1.0f, v_aliases_k != 0)) return rc;
    backward_balance(p, d_qk, d_v, v_aliases_k != 0);
    if (n_chunks) *n_chunks = p.n_split_kt > 0 ? p.split_chunks : 1;
    if (n_whole) *n_whole = ((int64_t)p.split_kt0() * p.max_chunks + (S + 63) / 64 - p.split_kt0() - p.n_split_kt) * Hkv * B;
    return p.n_split_kt;
}

int loza_ssa_backward(const void *q, const void *k, const void *v, const void *out, const float *lse,
                      const void *dout, void *dq, void *dk, void *dv,
                      int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                      int64_t n_sink, int64_t window, float scale,
                      void *workspace, size_t workspace_bytes, void *stream)
{
    return backward_bf16(q, k, v, out, lse, dout, dq, dk, dv, B, Hq, Hkv, S, d_qk, d_v, n_sink, window, 1, false, scale,
                         workspace, workspace_bytes, stream);
}

int loza_ssa_backward_blocks(const void *q, const void *k, const void *v, const void *out, const float *lse,
                             const void *dout, void *dq, void *dk, void *dv,
                             int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                             int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale,
                             void *workspace, size_t workspace_bytes, void *stream)
{
    return backward_bf16(q, k, v, out, lse, dout, dq, dk, dv, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block,
                         true, scale, workspace, workspace_bytes, stream);
}

static int backward_f32(const float *q, const float *k, const float *v, const float *out, const float *lse, const float *dout,
                        float *dq, float *dk, float *dv, int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                        int64_t sink, int64_t local, int64_t block, bool blocks, float scale, void *stream)
{
    if (!q || !k || !v || !out || !lse || !dout || !dq || !dk) return LOZA_ERR_NULL;
    if (int rc = check_common(B, Hq, Hkv, S, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    const bool alias = (v == k);
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (!alias && !dv) return LOZA_ERR_NULL;
    if (d_qk > 256 || d_v > 256) return LOZA_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse) || !aligned16(dout) ||
        !aligned16(dq) || !aligned16(dk) || (!alias && !aligned16(dv)))
        return LOZA_ERR_ALIGN;
    if (((int64_t)B * S * Hq + 3) / 4 > 2147483647LL) return LOZA_ERR_SHAPE;

    loza::F32BwdParams p{};
    p.q = q; p.k = k; p.v = v; p.out = out; p.lse = lse; p.dout = dout;
    p.dq = dq; p.dk = dk; p.dv = alias ? nullptr : dv;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.S = S; p.d_qk = d_qk; p.d_v = d_v;
    p.k_row = d_qk; p.v_row = alias ? d_qk : d_v;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S) : token_pattern(sink, local, S);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale = scale;
    return loza::launch_backward_f32(p, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_backward_f32(const float *q, const float *k, const float *v, const float *out, const float *lse,
                          const float *dout, float *dq, float *dk, float *dv,
                          int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                          int64_t n_sink, int64_t window, float scale, void *stream)
{
    return backward_f32(q, k, v, out, lse, dout, dq, dk, dv, B, Hq, Hkv, S, d_qk, d_v, n_sink, window, 1, false, scale, stream);
}

int loza_ssa_backward_blocks_f32(const float *q, const float *k, const float *v, const float *out, const float *lse,
                                 const float *dout, float *dq, float *dk, float *dv,
                                 int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                 int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale, void *stream)
{
    return backward_f32(q, k, v, out, lse, dout, dq, dk, dv, B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true,
                        scale, stream);
}

size_t loza_ssa_backward_workspace_bytes(int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                         int64_t n_sink, int64_t window, int v_aliases_k)
{
    return backward_workspace(B, Hq, Hkv, S, d_qk, d_v, n_sink, window, 1, false, v_aliases_k);
}

size_t loza_ssa_backward_workspace_bytes_blocks(int B, int Hq, int Hkv, int64_t S, int d_qk, int d_v,
                                                int64_t sink_blocks, int64_t local_blocks, int64_t block,
                                                int v_aliases_k)
{
    if (check_blocks(sink_blocks, local_blocks, block) != LOZA_OK) return 0;
    return backward_workspace(B, Hq, Hkv, S, d_qk, d_v, sink_blocks, local_blocks, block, true, v_aliases_k);
}

int loza_ssa_decode_num_splits(int B, int Hq, int Hkv, int64_t S_max, int64_t n_sink, int64_t window)
{
    if (check_common(B, Hq, Hkv, S_max, 1, 1, n_sink, window, 1.0f) != LOZA_OK) return 0;
    return decode_splits(B, Hq, Hkv, S_max, n_sink, window);
}

size_t loza_ssa_decode_workspace_bytes(int B, int Hq, int Hkv, int64_t S_max, int d_v,
                                       int64_t n_sink, int64_t window)
{
    if (d_v < 1) return 0;
    const int n = loza_ssa_decode_num_splits(B, Hq, Hkv, S_max, n_sink, window);
    if (n == 0) return 0;
    return (size_t)B * Hq * n * ((size_t)d_v + 4) * sizeof(float);
}

int loza_ssa_decode_kernel(int B, int Hq, int Hkv, int64_t S_max, int d_qk,
                           int64_t sink_blocks, int64_t local_blocks, int64_t block, int *n_splits)
{
    if (int rc = check_common(B, Hq, Hkv, S_max, d_qk, 1, sink_blocks, local_blocks, 1.0f)) return rc;
    if (int rc = check_blocks(sink_blocks, local_blocks, block)) return rc;
    if (!loza::bf16_width_supported(d_qk)) return LOZA_ERR_UNSUPPORTED;
    const DecodePlan plan = decode_plan(B, Hq, Hkv, S_max, d_qk, sat_mul(sink_blocks, block), sat_mul(local_blocks, block));
    if (n_splits) *n_splits = plan.n_splits;
    return plan.rows ? LOZA_KERNEL_ROWS : LOZA_KERNEL_TILES;
}

static int decode_bf16(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens,
                       void *out, float *lse, int B, int Hq, int Hkv, int64_t S_max,
                       int d_qk, int d_v, int64_t sink, int64_t local, int64_t block, bool blocks, float scale,
                       void *workspace, size_t workspace_bytes, void *stream, const Paging *paging = nullptr)
{
    if (!q || !kcache || !vcache || !seqlens || !out || !lse) return LOZA_ERR_NULL;
    int page_shift = 0;
    if (paging) {
        if (int rc = check_paging(*paging, &page_shift, &S_max)) return rc;
    }
    if (int rc = check_common(B, Hq, Hkv, S_max, d_qk, d_v, sink, local, scale)) return rc;
    if (blocks) { if (int rc = check_blocks(sink, local, block)) return rc; }
    if (!(scale > 0.f)) return LOZA_ERR_SHAPE;
    // the split count and the workspace are sized by the token counts the pattern can reach
    const int64_t n_sink = blocks ? sat_mul(sink, block) : sink, window = blocks ? sat_mul(local, block) : local;
    const bool alias = (vcache == kcache);
    if (alias && d_v > d_qk) return LOZA_ERR_SHAPE;
    if (!loza::bf16_shape_supported(d_qk, d_v, alias)) return LOZA_ERR_UNSUPPORTED;
    const size_t need = loza_ssa_decode_workspace_bytes(B, Hq, Hkv, S_max, d_v, n_sink, window);
    if (!workspace || workspace_bytes < need) return LOZA_ERR_WORKSPACE;
    if (!aligned16(q) || !aligned16(kcache) || !aligned16(vcache) || !aligned16(out) || !aligned16(workspace) ||
        (reinterpret_cast<uintptr_t>(seqlens) & 3u) || (reinterpret_cast<uintptr_t>(lse) & 3u))
        return LOZA_ERR_ALIGN;
    const int G = Hq / Hkv;
    const int rows = loza::decode_rows_per_tile();
    const DecodePlan plan = decode_plan(B, Hq, Hkv, S_max, d_qk, n_sink, window);
    const int n_splits = plan.n_splits;
    const int64_t row_tiles = (G + rows - 1) / rows;
    if (row_tiles * Hkv * B * decode_splits(B, Hq, Hkv, S_max, n_sink, window) > 2147483647LL) return LOZA_ERR_SHAPE;

    loza::FwdParams p{};
    p.q = (const uint16_t *)q; p.k = (const uint16_t *)kcache; p.v = (const uint16_t *)vcache;
    p.out = (uint16_t *)out; p.lse = lse;
    p.part_o = (float *)workspace;
    p.part_ml = (float *)workspace + (size_t)B * Hq * n_splits * d_v;
    p.seqlens = seqlens;
    if (paging) {
        p.block_table = paging->block_table;
        p.page_shift = page_shift; p.max_pages = paging->max_pages; p.num_pages = (int)paging->num_pages;
    }
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.G = G; p.S = S_max;
    const Pattern pat = blocks ? block_pattern(sink, local, block, S_max) : token_pattern(sink, local, S_max);
    p.n_sink = pat.n_sink; p.window = pat.window; p.block = pat.block;
    p.scale_log2 = scale * 1.44269504088896340736f;
    p.row_tiles = (int)row_tiles; p.n_splits = n_splits;
    set_rescale_policy(p);
    if (plan.rows) {
        p.q_len = 1;
        return loza::launch_rows_bf16(p, d_qk, d_v, alias, true, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
    }
    return loza::launch_decode_bf16(p, d_qk, d_v, alias, (hipStream_t)stream) == hipSuccess ? LOZA_OK : LOZA_ERR_HIP;
}

int loza_ssa_decode(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens,
                    void *out, float *lse, int B, int Hq, int Hkv, int64_t S_max,
                    int d_qk, int d_v, int64_t n_sink, int64_t window, float scale,
                    void *workspace, size_t workspace_bytes, void *stream)
{
    return decode_bf16(q, kcache, vcache, seqlens, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, n_sink, window, 1, false,
                       scale, workspace, workspace_bytes, stream);
}

int loza_ssa_decode_static(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens,
                           void *out, float *lse, int B, int Hq, int Hkv, int64_t S_max,
                           int d_qk, int d_v, int64_t n_sink, int64_t window, float scale, void *stream)
{
    // sizes first (no HIP call on a rejected size), then the per-device address of the scratch array
    if (check_common(B, Hq, Hkv, S_max, d_qk, d_v, n_sink, window, scale) != LOZA_OK) return LOZA_ERR_SHAPE;
    const size_t need = loza_ssa_decode_workspace_bytes(B, Hq, Hkv, S_max, d_v, n_sink, window);
    if (need == 0) return LOZA_ERR_SHAPE;
    if (need > (size_t)LOZA_DECODE_STATIC_BYTES) return LOZA_ERR_WORKSPACE;
    void *ws = nullptr;
    if (int rc = scratch_of_current_device(&ws)) return rc;
    return decode_bf16(q, kcache, vcache, seqlens, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, n_sink, window, 1, false,
                       scale, ws, (size_t)LOZA_DECODE_STATIC_BYTES, stream);
}

int loza_ssa_decode_paged(const void *q, const void *k_pages, const void *v_pages, const int32_t *block_table,
                          const int32_t *seqlens, void *out, float *lse, int B, int Hq, int Hkv,
                          int64_t num_pages, int page_size, int max_pages_per_seq, int d_qk, int d_v,
                          int64_t n_sink, int64_t window, float scale,
                          void *workspace, size_t workspace_bytes, void *stream)
{
    const Paging pg{block_table, num_pages, page_size, max_pages_per_seq};
    return decode_bf16(q, k_pages, v_pages, seqlens, out, lse, B, Hq, Hkv, 1, d_qk, d_v, n_sink, window, 1, false,
                       scale, workspace, workspace_bytes, stream, &pg);
}

int loza_ssa_decode_paged_blocks(const void *q, const void *k_pages, const void *v_pages, const int32_t *block_table,
                                 const int32_t *seqlens, void *out, float *lse, int B, int Hq, int Hkv,
                                 int64_t num_pages, int page_size, int max_pages_per_seq, int d_qk, int d_v,
                                 int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    const Paging pg{block_table, num_pages, page_size, max_pages_per_seq};
    return decode_bf16(q, k_pages, v_pages, seqlens, out, lse, B, Hq, Hkv, 1, d_qk, d_v, sink_blocks, local_blocks,
                       block, true, scale, workspace, workspace_bytes, stream, &pg);
}

int loza_ssa_decode_blocks(const void *q, const void *kcache, const void *vcache, const int32_t *seqlens,
                           void *out, float *lse, int B, int Hq, int Hkv, int64_t S_max,
                           int d_qk, int d_v, int64_t sink_blocks, int64_t local_blocks, int64_t block, float scale,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    return decode_bf16(q, kcache, vcache, seqlens, out, lse, B, Hq, Hkv, S_max, d_qk, d_v, sink_blocks, local_blocks,
                       block, true, scale, workspace, workspace_bytes, stream);
}

}  // extern "C"
