// Backward of bf16 streaming sparse attention, heads of width 128 (gfx950): dQ, and dK and dV.
//
// Same operation, work items and workspace as ssa_bwd.hip, which keeps the absorbed-MLA shape. There the four waves of
// a workgroup hand S, T, dS and p to each other through LDS behind three barriers per 32 x 64 tile; at this width a tile
// has so little matrix work (48 or 64 instructions for four waves) that the hand-over was most of its time: 1478 cycles
// per tile and compute unit for 384 of matrix work (dQ), 1570 for 512 (dK, dV). Here
//   * a wave owns 32 items X of the stationary side (query rows, or keys) through everything: S^T[32 y][32 x] = Y1 X1^T
//     and T^T = Y2 X2^T leave lane (h, n) with item n's values at y = 8 a + 4 h + 0 .. 3, and the order of the
//     contraction over y is free, so the eight dS (and p) a lane forms for 16 y are its B operand of Acc^T[d][x] +=
//     Y^T dS, whose A operand the transposing reads fetch in that order: nothing goes back to LDS;
//   * two waves per SIMD, of workgroups that do not wait for each other: one's matrix instructions run while the other
//     forms exponentials or waits for LDS. (A wave of 64 items would read half as much from LDS per matrix instruction,
//     but fill the register file alone, and overlap only what is interleaved by hand.)
//   * every wave reads the streamed tile twice, by rows and transposed; matrix and vector work in turn bound it (LDS busy
//     30 % of the cycles, matrix cores 59 and 59 %).
// 32 heads of their own keys, 8,111 tokens of 128 + 4096: dQ 1008 -> 600 us, dK and dV 1168 -> 830.
// Tiles of 32 items travel global -> LDS by global_load_lds_dwordx4; rows of 256 bytes are unpadded, their 16-byte
// chunks permuted (row_swizzle): both kinds of reads are free of bank conflicts. (By c ^ (r & 7) within groups of eight
// two thirds of the LDS's cycles were conflicts, and it was busy 71 and 73 % of the time; forward and backward of
// that case 1973 us, now 1891.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ssa_bwd_items.h"
#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One global -> LDS copy instruction (1 KB), unknown to the compiler's wait counters: the loop waits with explicit counts.
__device__ __forceinline__ void copy_1k(const char *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// pack_bf16 in one instruction (of values that a mask has chosen the compiler makes two and a permutation)
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Three bf16 terms that add up to x (all 24 bits), as a matrix operand's first three features. An infinity has no
// remainder.
__device__ __forceinline__ u32x2 three_terms(float x)
{
    const uint32_t w = pack2(x, 0.f);
    const float r = __builtin_fabsf(x) == __builtin_inff() ? 0.f : x - __builtin_bit_cast(float, w << 16);
    const uint32_t w2 = pack2(r, 0.f);
    u32x2 t;
    t[0] = w | w2 << 16;
    t[1] = pack2(r - __builtin_bit_cast(float, w2 << 16), 0.f);
    return t;
}

template <int N>
__device__ __forceinline__ void wait_copies()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

}  // namespace

template <bool ALIAS, bool KEYS>
struct Bwd128Cfg {
    static constexpr int D = 128, ROW = D * 2;
    // Four waves, two workgroups a compute unit. dQ: 128 rows, a tile a step. dK, dV: a work item of 64 keys, two tiles
    // a step, one for either pair of waves, whose sums meet in LDS at the end (with two waves a work item, the same
    // work in four workgroups a compute unit, few items left most of the chip idle: 8 key heads, 768 tokens 132 us, now 102).
    static constexpr int NW = 4, PAIRS = KEYS ? 2 : 1, X = NW / PAIRS * 32, PER_CU = 2;
    static constexpr bool HAS_Y2 = KEYS || !ALIAS;       // a second streamed tile (dO rows, or separate values)
    static constexpr bool SPLIT_KV = KEYS && !ALIAS;     // accumulators of dK and dV apart
    static constexpr int TILE = 32 * ROW;
    static constexpr int OFF_STAT = HAS_Y2 ? 2 * TILE : TILE;   // KEYS: 32 records of a row's statistics
    static constexpr int TSTAGE = OFF_STAT + (KEYS ? 1024 : 0), STAGE = PAIRS * TSTAGE;
    static constexpr int NST = KEYS ? 2 : 4;
    static constexpr int CP = 8 / NW * (HAS_Y2 ? 2 : 1) * PAIRS; // copy instructions per wave and stage (and one of waves 0, 1: the statistics)
    static constexpr int OUTROW = ROW + 16;              // LDS bytes per finished row
    // dK, dV: two accumulators, two operands and the tile's S and T leave a wave of 256 registers four short; the last
    // fragment of V waits in LDS (in scratch memory it would be a vector load that drains the copies under way)
    static constexpr int OFF_PARK = NST * STAGE, PARK = SPLIT_KV ? NW * 1024 : 0;
    static constexpr int LDS_BYTES = OFF_PARK + PARK > X * OUTROW ? OFF_PARK + PARK : X * OUTROW;
    static_assert(LDS_BYTES >= (KEYS ? (SPLIT_KV ? 2 : 1) * 2 * 64 * 256 : 0), "the results' way out");
    static_assert(LDS_BYTES * PER_CU <= 160 * 1024, "workgroups of a compute unit share the 160 KB LDS");
};

template <bool ALIAS, bool KEYS>
__global__ __launch_bounds__(256, 2) void ssa_bwd128_kernel(const BwdParams p)
{
    using C = Bwd128Cfg<ALIAS, KEYS>;
    constexpr int D = C::D, ROW = C::ROW, NST = C::NST, AHEAD = NST - 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, lh = lane >> 5;
    const int G = p.G;
    const int64_t S = p.S, R = S * G;
    const int n_sink = p.n_sink, window = p.window, block = p.block;
    const int g_log2 = (G & (G - 1)) == 0 ? __builtin_ctz((unsigned)G) : -1;
    auto div_g = [&](int r) { return g_log2 >= 0 ? r >> g_log2 : r / G; };

    // ---- which work item, and the streamed tiles of it ------------------------------------------------
    BwdItem it;
    int nt, nA = 0, nB = 0, wt0 = 0, w_rot = 0;
    int wi_min = 0, wi_max = 0, w_lo_min = 0, w_lo_max = 0;   // !KEYS: positions of this wave's rows, their windows' starts
    if constexpr (!KEYS) {
        // every XCD takes one contiguous eighth of the row tiles (they share most of their keys), heaviest first
        const int tiles = (int)((R + C::X - 1) / C::X);
        int id = blockIdx.x;
        const int eighth = gridDim.x / 8;
        if (id < eighth * 8) id = (id % 8) * eighth + id / 8;
        it.xt = tiles - 1 - id % tiles;
        id /= tiles;
        it.g = id % p.Hkv;
        it.b = id / p.Hkv;
        const int64_t r0 = (int64_t)it.xt * C::X, w0 = r0 + wave * 32 < R ? r0 + wave * 32 : R - 1;
        const int i_min = (int)row_position(r0, G), i_max = (int)row_position(r0 + C::X - 1 < R ? r0 + C::X - 1 : R - 1, G);
        wi_min = (int)row_position(w0, G);
        wi_max = (int)row_position(w0 + 31 < R ? w0 + 31 : R - 1, G);
        w_lo_min = window_begin_of(wi_min, window, block);
        w_lo_max = window_begin_of(wi_max, window, block);
        const int sink_end = n_sink < i_max + 1 ? n_sink : i_max + 1;
        nA = (sink_end + 31) / 32;
        wt0 = window_begin_of(i_min, window, block) / 32;
        const int wt1 = i_max / 32;
        if (wt0 <= nA) nA = wt1 + 1;
        else nB = wt1 - wt0 + 1;
        nt = nA + nB;
        // (window tiles in rotated order: row tiles that run together ask for the same keys at the same step)
        if (nB > 1) { w_rot = wt0 % nB; w_rot = w_rot == 0 ? 0 : nB - w_rot; }
    } else {
        it = bwd_key_item(p, blockIdx.x);
        nt = it.nt;
        if (nt <= 0) return;   // a chunk beyond the rows of this key tile (the reduce kernel knows)
    }
    const int b = it.b, g = it.g;
    // first item of streamed tile t
    auto y_first = [&](int t) {
        if constexpr (KEYS) {
            const int yt = it.yt_start + t;
            return (yt < it.yt_begin + it.nt ? yt : yt - it.nt) * 32;
        } else {
            if (t < nA) return t * 32;
            int x = t - nA + w_rot;
            x = x >= nB ? x - nB : x;
            return (wt0 + x) * 32;
        }
    };

    // ---- copies: instruction n of a sub-tile's eight moves rows 4 n .. 4 n + 3 and belongs to wave n % NW --------
    const int n_y = (int)(KEYS ? R : S);
    const int c_row = wave * 4 + (lane >> 4);
    const uint32_t c_chunk = ((uint32_t)(lane & 15) ^ row_swizzle(c_row)) * 16u;   // (a wave's rows are equal mod 16)
    // byte offset of row y of a tile from its first row
    auto item_offset = [&](int y) -> uint32_t {
        if (!KEYS) return (uint32_t)y * (uint32_t)p.Hkv * ROW;
        if (G >= 32) return (uint32_t)y * ROW;                                      // 32 heads of one position
        const int i = y >> g_log2;
        return (uint32_t)(i * p.Hq + (y - (i << g_log2))) * ROW;
    };
    // (a wave's rows c_row and c_row + 16 lie the same distance apart in every lane, of 16 heads a position or fewer as of
    // more; registers are short, so one offset a lane)
    constexpr int NX = 8 / C::NW, STEP = C::NW * 4;
    const uint32_t off0 = item_offset(c_row) + c_chunk;
    uint32_t step_off[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) step_off[x] = item_offset(x * STEP);
    const uint32_t full = item_offset(31) + ROW - 16;
    const char *y1_all = (const char *)(KEYS ? p.q : p.k), *y2_all = (const char *)(KEYS ? p.dout : p.v);
    const int64_t row_base = KEYS ? (int64_t)b * S * p.Hq + (int64_t)g * G : (int64_t)b * S * p.Hkv + g;
    const float2 *stats = p.rowstat + ((int64_t)b * p.Hkv + g) * p.r_pad;
    auto copy_one = [&](int t, uint32_t stage, int half) {
        const int y0 = y_first(t);
        const int64_t row0 = KEYS ? row_base + y0 + (int64_t)div_g(y0) * (p.Hq - G) : row_base + (int64_t)y0 * p.Hkv;
        const char *b1 = y1_all + row0 * ROW, *b2 = y2_all + row0 * ROW;
        const uint32_t dst = stage + half * C::TSTAGE + wave * 1024;
        // (in the ragged last tile what lies past the last item is cut to its last chunk)
        const uint32_t last = y0 + 31 < n_y ? full : item_offset(n_y - 1 - y0) + ROW - 16;
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const uint32_t o = off0 + step_off[x] < last ? off0 + step_off[x] : last;
            copy_1k(b1, o, dst + x * C::NW * 1024);
            if (C::HAS_Y2) copy_1k(b2, o, dst + C::TILE + x * C::NW * 1024);
        }
        if (KEYS && wave == half) copy_1k((const char *)(stats + y0), (uint32_t)(lane & 15) * 16u, stage + half * C::TSTAGE + C::OFF_STAT);
    };
    // step u: tiles PAIRS u, ... (past the last tile, that one again: the wait counts are the same throughout)
    auto copy_step = [&](int u, int st) {
#pragma unroll
        for (int half = 0; half < C::PAIRS; ++half) copy_one(u * C::PAIRS + half < nt ? u * C::PAIRS + half : nt - 1, smem_lds + st * C::STAGE, half);
    };
    const int pair = KEYS ? wave >> 1 : 0, xb = KEYS ? wave & 1 : wave;             // which tile of a step, which 32 items

    // ---- the stationary side: matrix-core B operands, item ln of this wave's block ----------------------
    bf16x8 x1[8], x2[ALIAS && KEYS ? 1 : 8];
    const int x_idx = it.xt * C::X + xb * 32 + ln;                                  // (S G <= 2^31 - 65: the last of 128 rows is 2^31 - 1 at most)
    const int64_t x_c = x_idx < (KEYS ? S : R) ? x_idx : (KEYS ? S : R) - 1;
    int x_i = 0;                                                                    // !KEYS: position of this lane's row
    float x_lse2 = 0.f, x_D = 0.f;                                                  // - lse log2(e), - D
    {
        int64_t row;
        if constexpr (!KEYS) {
            const int64_t i = row_position(x_c, G);
            x_i = (int)i;
            row = ((int64_t)b * S + i) * p.Hq + (int64_t)g * G + (x_c - i * G);
            const float2 st = stats[x_c];
            x_lse2 = -st.x;
            x_D = -st.y;
        } else {
            row = ((int64_t)b * S + x_c) * p.Hkv + g;
        }
        const uint16_t *p1 = (KEYS ? p.k : p.q) + row * D + lh * 8, *p2 = (KEYS ? p.v : p.dout) + row * D + lh * 8;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            x1[kk] = *(const bf16x8 *)(p1 + kk * 16);
            if constexpr (!(ALIAS && KEYS)) x2[kk] = *(const bf16x8 *)(p2 + kk * 16);
        }
    }
    const int w_lo_row = KEYS ? 0 : window_begin_of(x_i, window, block);
    // (waited for with a wait the compiler sees: left to its own bookkeeping it would wait for them inside the loop,
    // with counts that also drain the tile copies it does not know about)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        asm volatile("" : "+v"(x1[kk]));
        if constexpr (!(ALIAS && KEYS)) {
            if (!C::SPLIT_KV || kk < 7) asm volatile("" : "+v"(x2[kk]));
        }
    }
    const uint32_t park = smem_lds + C::OFF_PARK + wave * 1024 + lane * 16;
    if constexpr (C::SPLIT_KV) *(__attribute__((address_space(3))) bf16x8 *)(uintptr_t)park = x2[7];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) copy_step(a, a);

    constexpr int NACC = C::SPLIT_KV ? 2 : 1;
    f32x16 acc[NACC][4];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][db][e] = 0.f;

    // LDS offsets of this lane's reads within a tile (by rows: row ln; transposing: rows 4 lh + ...)
    // (of fragment 0; the permutation makes the others' a matter of single bits: tiles lie at multiples of 1 KB)
    const int s16 = lane & 15, v_row = lh * 4 + (s16 >> 2);
    const uint32_t k_rd = (uint32_t)(ln * ROW) + ((uint32_t)lh ^ row_swizzle(ln)) * 16u;
    const uint32_t v_rd = (uint32_t)(v_row * ROW + (s16 & 1) * 8) + ((uint32_t)(((lane >> 4) & 1) * 2 + ((s16 & 3) >> 1)) ^ row_swizzle(v_row)) * 16u;
    typedef __attribute__((address_space(3))) const char *lds_ptr;
    auto read_rows = [&](uint32_t t, int kk) {
        return *(__attribute__((address_space(3))) const bf16x8 *)(uintptr_t)(t ^ (kk << 5));
    };
    auto read_cols = [&](uint32_t t, int ks, int db) {
        const lds_ptr a = (lds_ptr)(uintptr_t)((t ^ (db << 6)) + ks * 16 * ROW), c = (lds_ptr)(uintptr_t)((t ^ (db << 6 | 32)) + ks * 16 * ROW + 8 * ROW);   // (row r + 8: swizzled by 2 more)
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(c));
        s16x8 a8;
        a8[0] = lo[0]; a8[1] = lo[1]; a8[2] = lo[2]; a8[3] = lo[3];
        a8[4] = hi[0]; a8[5] = hi[1]; a8[6] = hi[2]; a8[7] = hi[3];
        return __builtin_bit_cast(bf16x8, a8);
    };

    constexpr int PF = C::SPLIT_KV ? 3 : 6;
    // ---- one tile of 32 y ----------------------------------------------------------------------------------
    // KEYS: the rows that see key j are the run [j G, last_row(j)]: the window's start does not decrease with the position
    auto last_row = [&](int64_t j) -> int {
        if (j < n_sink) return (int)R - 1;
        const int64_t r = ((j / block + window) * (int64_t)block) * G - 1;
        return r < R ? (int)r : (int)R - 1;
    };
    int y_lo = 0, y_hi = 0;                                                         // of this lane's key
    const float to_score = -1.0f / p.scale_log2;                                    // lse log2(e) -> - lse in units of the scores
    int any_lo = 0, any_hi = 0, all_lo = 0, all_hi = 0;                             // of some, of all of the wave's keys
    if constexpr (KEYS) {
        const int64_t kj0 = (int64_t)it.xt * C::X + xb * 32, kj1 = kj0 + 31;
        y_lo = x_idx < S ? x_idx * G : 0x7fffffff;
        y_hi = last_row(x_idx);
        any_lo = kj0 < S ? (int)(kj0 * G) : 0x7fffffff;
        any_hi = kj0 < n_sink ? (int)R - 1 : last_row(kj1);
        all_lo = kj1 < S ? (int)(kj1 * G) : 0x7fffffff;
        all_hi = kj1 < n_sink ? (int)R - 1 : last_row(kj0 < n_sink ? (int64_t)n_sink : kj0);
    }
    auto tile_step = [&](const int y0, const uint32_t t1) {
        constexpr uint32_t SECOND = C::HAS_Y2 ? C::TILE : 0;
        bool dead, interior;                                                        // of this wave's 32 x 32 pairs
        if constexpr (!KEYS) {
            dead = y0 > wi_max || (y0 >= n_sink && y0 + 31 < w_lo_min);
            interior = y0 + 31 <= wi_min && (y0 + 31 < n_sink || y0 >= w_lo_max);
        } else {
            dead = y0 + 31 < any_lo || y0 > any_hi;
            interior = y0 >= all_lo && y0 + 31 <= all_hi;
        }
        if (dead) return;
        // (matrix phases first: the waves of the other workgroups fill in; 3 % of dQ)
        __builtin_amdgcn_s_setprio(1);
        f32x16 s, t;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; t[e] = 0.f; }
        {
            // (fragments PF steps ahead; the scheduling barriers keep the compiler from fetching all of them at once,
            // for registers it does not have)
            bf16x8 f[PF], parked;
            uint32_t a1 = t1 + k_rd;
            asm volatile("" : "+v"(a1));
            auto fetch = [&](int m) { return m < 8 ? read_rows(a1, m) : read_rows(a1 + SECOND, m - 8); };
            if constexpr (KEYS) {
                // The rows' - lse / scale and - D, three bf16 terms each, are one more step of either contraction
                // (read as they are, 16 values a lane, they were a third of this phase's LDS time). The second half
                // of the wave, whose part of the contraction is empty, takes zeros.
                const f32x2 rec = *(__attribute__((address_space(3))) const f32x2 *)(uintptr_t)(t1 + C::OFF_STAT + ln * 8);
                auto add = [&](float v, f32x16 &x) {
                    const u32x2 t3 = three_terms(v);
                    const u32x4 terms = {lh == 0 ? t3[0] : 0, lh == 0 ? t3[1] : 0, 0, 0}, ones = {0x3f803f80u, 0x3f80u, 0, 0};
                    x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, terms), __builtin_bit_cast(bf16x8, ones), x, 0, 0, 0);
                };
                add(rec[0] * to_score, s);
                add(-rec[1], t);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int m = 0; m < PF; ++m) f[m] = fetch(m);
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                if (m < 8) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m % PF], x1[m], s, 0, 0, 0);
                else if (m < 15 || !C::SPLIT_KV) t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m % PF], ALIAS && KEYS ? x1[m - 8] : x2[m - 8], t, 0, 0, 0);
                else t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m % PF], parked, t, 0, 0, 0);
                if (C::SPLIT_KV && m == 12) parked = *(__attribute__((address_space(3))) const bf16x8 *)(uintptr_t)park;
                if (m + PF < 16) f[m % PF] = fetch(m + PF);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        u32x4 pb[KEYS ? 2 : 1], sb[2];
        __builtin_amdgcn_s_setprio(0);
        auto elementwise = [&](auto masked_c) {
            constexpr bool MASKED = decltype(masked_c)::value;
#pragma unroll
            for (int a = 0; a < 4; ++a) {                                           // y = 8 a + 4 lh + 0 .. 3
                float pv[4], ds[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bool ok = true;
                    if constexpr (MASKED && !KEYS) {
                        const int j = y0 + 8 * a + 4 * lh + e;
                        ok = (j <= x_i) & ((j < n_sink) | (j >= w_lo_row));
                    }
                    if constexpr (MASKED && KEYS) {
                        const int y = y0 + 8 * a + 4 * lh + e;
                        ok = (y >= y_lo) & (y <= y_hi);
                    }
                    const float pe = __builtin_amdgcn_exp2f(KEYS ? s[4 * a + e] * p.scale_log2 : __builtin_fmaf(s[4 * a + e], p.scale_log2, x_lse2));
                    const float de = (C::SPLIT_KV || !KEYS ? pe : p.scale * pe) * (KEYS ? t[4 * a + e] : t[4 * a + e] + x_D);
                    pv[e] = ok ? pe : 0.f;
                    ds[e] = ok ? de : 0.f;
                }
                sb[a >> 1][(a & 1) * 2] = pack2(ds[0], ds[1]);
                sb[a >> 1][(a & 1) * 2 + 1] = pack2(ds[2], ds[3]);
                if constexpr (KEYS) {
                    pb[a >> 1][(a & 1) * 2] = pack2(pv[0], pv[1]);
                    pb[a >> 1][(a & 1) * 2 + 1] = pack2(pv[2], pv[3]);
                }
            }
        };
        if (interior) elementwise(std::false_type{});
        else {
            asm volatile("");   // (a branch, no predicate in the path that needs none)
            elementwise(std::true_type{});
        }
        {
            __builtin_amdgcn_s_setprio(1);
            constexpr int PROD = KEYS ? 2 : 1, NF = 8 * PROD;                       // (products: dS with Y1, p with Y2)
            bf16x8 f[PF];
            uint32_t a1 = t1 + v_rd;
            asm volatile("" : "+v"(a1));
            auto fetch = [&](int m) { return read_cols(m % PROD ? a1 + SECOND : a1, m / PROD >> 2, m / PROD & 3); };
#pragma unroll
            for (int m = 0; m < PF; ++m) f[m] = fetch(m);
#pragma unroll
            for (int m = 0; m < NF; ++m) {
                const int ks = m / PROD >> 2, db = m / PROD & 3;
                const u32x4 w = m % PROD ? pb[KEYS ? ks : 0] : sb[ks];
                f32x16 &x = acc[m % PROD ? NACC - 1 : 0][db];
                x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m % PF], __builtin_bit_cast(bf16x8, w), x, 0, 0, 0);
                if (m + PF < NF) f[m % PF] = fetch(m + PF);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
        }
    };

    int st = 0;
    for (int u = 0; u * C::PAIRS < nt; ++u) {
        // step u has landed when at most the copies of the steps after it are outstanding
        if (KEYS && wave < 2) wait_copies<(AHEAD - 1) * (C::CP + 1)>();
        else wait_copies<(AHEAD - 1) * C::CP>();
        lds_barrier();                                                              // ... everyone's; step u - 1 is no longer read
        copy_step(u + AHEAD, st == 0 ? NST - 1 : st - 1);
        if (u * C::PAIRS + pair < nt) tile_step(y_first(u * C::PAIRS + pair), smem_lds + st * C::STAGE + pair * C::TSTAGE);
        st = st + 1 < NST ? st + 1 : 0;
    }
    wait_copies<0>();                                                               // (nothing may be on its way into LDS any more)
    lds_barrier();

    // ---- results ---------------------------------------------------------------------------------------------
    if constexpr (KEYS) {
        const uint32_t sums = smem_lds + xb * (NACC * 64 * 256) + lane * 16;
        if (pair == 1) {
#pragma unroll
            for (int a = 0; a < NACC; ++a)
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd)
                        *(__attribute__((address_space(3))) f32x4 *)(uintptr_t)(sums + ((a * 4 + db) * 4 + qd) * 1024) =
                            f32x4{acc[a][db][4 * qd], acc[a][db][4 * qd + 1], acc[a][db][4 * qd + 2], acc[a][db][4 * qd + 3]};
        }
        lds_barrier();
        if (pair == 1) return;
#pragma unroll
        for (int a = 0; a < NACC; ++a)
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int qd = 0; qd < 4; ++qd) {
                    const f32x4 v = *(__attribute__((address_space(3))) const f32x4 *)(uintptr_t)(sums + ((a * 4 + db) * 4 + qd) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[a][db][4 * qd + e] += v[e];
                }
        if (it.partial) {
            // row [dK | dV (separate values only)] of fp32 partial sums
            constexpr int COLS = C::SPLIT_KV ? 2 * D : D;
            float *op = p.part + (it.slot * 64 + xb * 32 + ln) * COLS + 4 * lh;
            if (x_idx >= S) return;
#pragma unroll
            for (int a = 0; a < NACC; ++a)
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) {
                        const float f = C::SPLIT_KV && a == 0 ? p.scale : 1.f;
                        float4 w;
                        w.x = acc[a][db][4 * qd] * f; w.y = acc[a][db][4 * qd + 1] * f; w.z = acc[a][db][4 * qd + 2] * f; w.w = acc[a][db][4 * qd + 3] * f;
                        *(float4 *)(op + a * D + db * 32 + qd * 8) = w;
                    }
            return;
        }
    }
    // this wave's 32 rows through LDS (its own part of it), then whole rows
    char *mine = smem + xb * (KEYS ? NACC * 64 * 256 : 32 * C::OUTROW);             // (KEYS: what this wave has just read)
#pragma unroll
    for (int a = 0; a < NACC; ++a) {
        const float f = !KEYS || (C::SPLIT_KV && a == 0) ? p.scale : 1.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                u32x2 w;
                w[0] = pack_bf16(acc[a][db][4 * qd] * f, acc[a][db][4 * qd + 1] * f);
                w[1] = pack_bf16(acc[a][db][4 * qd + 2] * f, acc[a][db][4 * qd + 3] * f);
                *(u32x2 *)(mine + ln * C::OUTROW + db * 64 + qd * 16 + lh * 8) = w;
            }
        uint16_t *base = !KEYS ? p.dq : a == 0 ? p.dk : p.dv;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int r = n * 4 + (lane >> 4);
            const int64_t x = (int64_t)it.xt * C::X + xb * 32 + r;
            const u32x4 w = *(const u32x4 *)(mine + r * C::OUTROW + (lane & 15) * 16);
            if (x >= (KEYS ? S : R)) continue;
            int64_t row;
            if constexpr (KEYS) {
                row = ((int64_t)b * S + x) * p.Hkv + g;
            } else {
                const int64_t i = row_position(x, G);
                row = ((int64_t)b * S + i) * p.Hq + (int64_t)g * G + (x - i * G);
            }
            *(u32x4 *)(base + row * D + (lane & 15) * 8) = w;
        }
    }
}

template <bool ALIAS, bool KEYS>
static hipError_t launch_t(const BwdParams &p, int64_t blocks, hipStream_t stream)
{
    using C = Bwd128Cfg<ALIAS, KEYS>;
    constexpr auto kern = ssa_bwd128_kernel<ALIAS, KEYS>;
    hipError_t e = allow_lds<kern>(C::LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * C::NW), C::LDS_BYTES, stream, p);
    return hipGetLastError();
}

// The key-stationary kernel works in units of the scores, where lse / scale has to be finite: a smaller scale is taken as
// 2^-100 in front of the scores (log-sum-exps up to 2^26 then are; the weights' exponents move by at most 2^-100 |q . k|).
hipError_t launch_bwd128_keys(BwdParams p, bool alias, int64_t items, hipStream_t stream)
{
    if (p.scale_log2 < 0x1p-100f) p.scale_log2 = 0x1p-100f;
    return alias ? launch_t<true, true>(p, items, stream) : launch_t<false, true>(p, items, stream);
}

hipError_t launch_bwd128_rows(const BwdParams &p, bool alias, hipStream_t stream)
{
    const int64_t tiles = (p.S * p.G + Bwd128Cfg<true, false>::X - 1) / Bwd128Cfg<true, false>::X * p.Hkv * p.B;
    return alias ? launch_t<true, false>(p, tiles, stream) : launch_t<false, false>(p, tiles, stream);
}

}  // namespace loza
