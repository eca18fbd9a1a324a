// Backward of the absorbed-MLA shape (576-wide keys whose first 512 columns are the values) in three passes, for gfx950.
//
// ssa_bwd.hip forms S = Q K^T and T = dO V^T twice, once for dQ and once for dK, and passes them between its waves
// through LDS behind three barriers per tile of 32 x 64: 3180 and 4850 cycles for 1664 and 2176 of matrix work. Here they
// are formed once and the weights p and dS, rounded to bf16 as there, go through memory:
//   * scores: a workgroup owns 128 query rows, its four waves 32 each with q and dO as matrix operands in registers
//     (272 of them), and walks the live key tiles of 32. The values are the key rows' prefix, so one fragment from LDS
//     feeds S and T both (36 reads for 68 matrix instructions); p and dS of a tile are formed between the matrix
//     instructions of the next one, and leave as fragments that the other passes take as operands;
//   * dQ: 128 rows, dQ^T[d][row] += K^T dS^T over the key tiles;
//   * dK and dV, one gradient here: 128 keys, dK^T[d][key] += Q^T dS + dO^T p over the row blocks of 32 that see them.
// The last two are matrix products and nothing else. Of the 128 x 576 results a wave holds 128 columns below 512 in all
// of its 256 accumulation registers, and of the last 64 columns the part of one block of 32 rows or keys in vector
// registers, so every transposed fragment of the streamed tile (16 cycles of LDS) feeds four matrix instructions.
// Memory: 4 bytes a pair and pass, written once and read by either product. Rows are taken in chunks whose weights fit the
// scratch memory that the host sets aside; a chunk's dK is cut into work items (128 keys x a segment of its rows), whose
// fp32 partial sums the reduction adds in order, onto those of the chunks before.
// 16,384 tokens, 64 heads, 1 + 7 blocks of 128 (rocprofv3): dK and dV 6.12 ms and dQ 3.57 before; now scores 2.37, dK and
// dV 2.6, dQ 1.4, reduction 0.1. Cycles: a scores tile 3050 for 2176 of matrix work (the stores 440), and 33 thousand of a
// row tile's 131 before its first: its 272 KB of q and dO, which all workgroups ask memory for together; 32 rows x 128
// keys of dK 3150 for 2240 (2490 without copies, 2650 where what they fetch is in L2: misses fill the memory pipeline's
// queue and the copy instructions wait for it), 32 keys x 128 rows of dQ 1720 for 1152.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "score_asm.h"
#include "ssa_bwd_tile.h"
#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

namespace {

constexpr int kDqk = 576, kDv = 512;
// Padded LDS rows. Read by rows, 16 bytes a lane: an odd number of 16-byte chunks, no bank conflicts. Read transposed only: 32
// bytes (a third to a half of the LDS's active cycles of the two products are conflicts; with 64 there are none, and the
// time is the same, 9,180 and 9,200 us forward and backward of the case below: LDS does not bound them).
constexpr int kPadT = 32;
constexpr int kRow1 = kDqk * 2 + 16, kRow1T = kDqk * 2 + kPadT, kRow2T = kDv * 2 + kPadT;
constexpr int kCopies1 = 37, kCopies1T = (32 * kRow1T + 1023) / 1024, kCopies2T = (32 * kRow2T + 1023) / 1024;   // 1 KB copies of a tile of 32 rows
static_assert(kCopies1 * 1024 >= 32 * kRow1 && (kCopies1T == 37 || kCopies1T == 38) && (kCopies2T == 33 || kCopies2T == 34), "copies cover the tile");
constexpr int kStageScores = kCopies1 * 1024, kOffB = kCopies1T * 1024, kStageProduct = kOffB + 8192;
constexpr int kLdsScores = 3 * kStageScores, kLdsProduct = 3 * kStageProduct;
constexpr int kRowOut = kDqk * 2 + 16, kLdsDq = kLdsProduct > 128 * kRowOut ? kLdsProduct : 128 * kRowOut;
static_assert(kLdsDq <= 160 * 1024, "does not fit the 160 KB LDS");
constexpr int64_t kBlockBytes = 16384;                       // weights of 32 rows x 128 keys: p of four key tiles, then dS

// Live keys of query rows [128 t, 128 t + 128) (t of row_tiles): as tiles of 32 and as groups of 128 keys.
struct RowTileKeys {
    int i_min, i_max, win_begin, sink_end;
    __device__ __forceinline__ RowTileKeys(const BwdParams &p, int64_t R, int64_t r0, int64_t r1)   // rows r0 .. r1 - 1
    {
        i_min = (int)row_position(r0, p.G);
        i_max = (int)row_position((r1 < R ? r1 : R) - 1, p.G);
        win_begin = window_begin_of(i_min, p.window, p.block);
        sink_end = p.n_sink < i_max + 1 ? p.n_sink : i_max + 1;
    }
    // tiles (or groups) of 2^shift keys: [0, nA) and nB from w0 on
    __device__ __forceinline__ void pieces(int shift, int &nA, int &w0, int &nB) const
    {
        const int w1 = i_max >> shift;
        nA = (sink_end + (1 << shift) - 1) >> shift;
        w0 = win_begin >> shift;
        if (w0 <= nA) { nA = w1 + 1; nB = 0; } else nB = w1 - w0 + 1;
    }
};

// Place of key group kg among the groups a row block can have: sinks first, the window's in a ring.
__device__ __forceinline__ int group_slot(const WideChunk &c, int kg)
{
    if (kg < c.sink_groups) return kg;
    return c.sink_groups + kg - c.win_groups * (int)__umulhi((uint32_t)kg, c.win_magic);
}

__device__ __forceinline__ char *weights_at(const WideChunk &c, int bgl, int rb, int kg)   // rb: row block of 32, of its (batch, key head)
{
    const int64_t row = (int64_t)bgl * (c.t1 - c.t0) * 4 + (rb - c.t0 * 4);
    return c.scratch + (row * c.slots + group_slot(c, kg)) * kBlockBytes;
}

// Byte offset within a tile of 32 items (consecutive items `stride` bytes apart) of what lane `lane` fetches with copy
// instruction n: slot n * 64 + lane of the padded tile is a chunk of 16 bytes; padding fetches a valid chunk.
template <int ROW, int DATA>
__device__ __forceinline__ uint32_t chunk_offset(int n, int lane, uint32_t (*item_offset)(int, uint32_t, uint32_t, int), uint32_t a, uint32_t b, int s)
{
    constexpr int CPR = ROW / 16;
    const int slot = n * 64 + lane, item = slot / CPR < 31 ? slot / CPR : 31, c = slot % CPR < DATA / 16 ? slot % CPR : DATA / 16 - 1;
    return item_offset(item, a, b, s) + c * 16;
}
__device__ __forceinline__ uint32_t key_item(int item, uint32_t stride, uint32_t, int) { return item * stride; }
// query rows: position-major, 2^s heads of a group together (s = 5 stands for more: one position's heads)
__device__ __forceinline__ uint32_t row_item(int item, uint32_t pos_stride, uint32_t head_stride, int s)
{
    return (item >> s) * pos_stride + (item & ((1 << s) - 1)) * head_stride;
}

// Row tiles of [ta, tb) that see a key of group kg: [see0, see1).
__device__ __forceinline__ void group_rows(const BwdParams &p, int kg, int ta, int tb, int &see0, int &see1)
{
    see0 = kg * p.G > ta ? kg * p.G : ta;
    see1 = tb;
    if (kg * 128 >= p.n_sink) {
        const int64_t i_w = ((int64_t)(kg * 128 + 127) / p.block + p.window) * p.block - 1, t_w = (i_w * p.G + p.G - 1) / 128 + 1;
        if (t_w < see1) see1 = (int)t_w;
    }
}

}  // namespace

// ---- scores: p and dS of 128 rows against their live keys ------------------------------------------------
__global__ __launch_bounds__(256) void ssa_bwd_wide_scores_kernel(const BwdParams p, const WideChunk c)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, lh = lane >> 5;
    const int G = p.G;
    const int64_t S = p.S, R = S * G;
    const int n_t = c.t1 - c.t0, bgl = blockIdx.x / n_t, t = c.t1 - 1 - blockIdx.x % n_t;   // latest (heaviest) rows first
    const int b = (c.bg0 + bgl) / p.Hkv, g = (c.bg0 + bgl) % p.Hkv;
    const int rb = t * 4 + wave;

    const RowTileKeys keys(p, R, (int64_t)t * 128, (int64_t)t * 128 + 128);
    int nA, wt0, nB;
    keys.pieces(5, nA, wt0, nB);
    const int nt = nA + nB;
    auto y_tile = [&](int u) { return u < nA ? u : wt0 + (u - nA); };
    const int w_lo_max = window_begin_of(keys.i_max, p.window, p.block);

    // matrix operands of this lane's row: q, then dO
    bf16x8 xf[kDqk / 16 + kDv / 16];
    {
        const int64_t row = (int64_t)rb * 32 + ln, r = row < R ? row : R - 1, i = row_position(r, G);
        const int64_t at = ((int64_t)b * S + i) * p.Hq + (int64_t)g * G + (r - i * G);
        const uint16_t *qp = p.q + at * kDqk + lh * 8, *dp = p.dout + at * kDv + lh * 8;
#pragma unroll
        for (int kk = 0; kk < kDqk / 16; ++kk) xf[kk] = *(const bf16x8 *)(qp + kk * 16);
#pragma unroll
        for (int kk = 0; kk < kDv / 16; ++kk) xf[kDqk / 16 + kk] = *(const bf16x8 *)(dp + kk * 16);
    }
    // statistics of the 16 rows whose values this lane gets: 8 (e / 4) + 4 lh + e % 4
    float lse2[16], dd[16];
    {
        const float2 *st = p.rowstat + (int64_t)(c.bg0 + bgl) * p.r_pad;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t row = (int64_t)rb * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
            const float2 v = st[row < R ? row : R - 1];
            lse2[e] = v.x;
            dd[e] = v.y;
        }
    }

    // key tiles of a group that this row tile sees, but none of whose keys do any of its rows: zeros
    {
        int gA, wg0, gB;
        keys.pieces(7, gA, wg0, gB);
        for (int x = 0; x < gA + gB; ++x) {
            const int kg = x < gA ? x : wg0 + (x - gA);
            char *blk = weights_at(c, bgl, rb, kg) + lane * 16;
            for (int k4 = 0; k4 < 4; ++k4) {
                const int kt = kg * 4 + k4;
                if (kt < nA || (kt >= wt0 && kt < wt0 + nB)) continue;
                const u32x4 z = {0, 0, 0, 0};
#pragma unroll
                for (int f = 0; f < 4; ++f) *(u32x4 *)(blk + (f >> 1) * 8192 + k4 * 2048 + (f & 1) * 1024) = z;
            }
        }
    }

    const uint32_t k_stride = (uint32_t)p.Hkv * (kDqk * 2);
    uint32_t voff[10];
#pragma unroll
    for (int x = 0; x < 10; ++x) voff[x] = chunk_offset<kRow1, kDqk * 2>(x < 9 ? x * 4 + wave : 36, lane, key_item, k_stride, 0, 0);
    const char *k_base = (const char *)(p.k + ((int64_t)b * S * p.Hkv + g) * kDqk);
    struct TileCopy { const char *src; uint32_t max, dst, dstx; };
    auto plan_tile = [&](int u, int stage) {
        const int y0 = y_tile(u < nt ? u : nt - 1) * 32, last = (int)S - 1 - y0 < 31 ? (int)S - 1 - y0 : 31;
        TileCopy tc;
        tc.src = k_base + (int64_t)y0 * k_stride;
        tc.max = last * k_stride + kDqk * 2 - 16;
        tc.dst = smem_lds + stage * kStageScores + wave * 1024;
        tc.dstx = smem_lds + stage * kStageScores + 36 * 1024;
        return tc;
    };
    auto copy_tile = [&](const TileCopy &tc) {
#pragma unroll
        for (int x = 0; x < 9; ++x) copy_1k(tc.src, voff[x] < tc.max ? voff[x] : tc.max, tc.dst + x * 4096);
        if (wave == 0) copy_1k(tc.src, voff[9] < tc.max ? voff[9] : tc.max, tc.dstx);
    };
    copy_tile(plan_tile(0, 0));
    copy_tile(plan_tile(1, 1));
    // (operands, statistics and the first tiles: with a wait that the compiler sees, or it waits for its own loads in the loop)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
    for (int kk = 0; kk < kDqk / 16 + kDv / 16; ++kk) {
        if (kk < 64) asm volatile("" : "+a"(xf[kk]));
        else asm volatile("" : "+v"(xf[kk]));
    }

    // Weights of tile u, packed in pairs of rows: mask what no row sees, store.
    auto put = [&](int u, uint32_t (&pw)[8], uint32_t (&dw)[8]) {
        const int kt = y_tile(u), y0 = kt * 32;
        const bool interior = y0 + 31 <= keys.i_min && (y0 + 31 < p.n_sink || y0 >= w_lo_max) && (int64_t)rb * 32 + 31 < R;
        if (!interior) {
            const int j = y0 + ln;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                uint32_t m = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int e = 2 * x + h;
                    const int64_t row = (int64_t)rb * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
                    const int i = (int)row_position(row, G);
                    const bool ok = (row < R) & (j <= i) & ((j < p.n_sink) | (j >= window_begin_of(i, p.window, p.block)));
                    m |= ok ? 0xffffu << (16 * h) : 0u;
                }
                pw[x] &= m;
                dw[x] &= m;
            }
        }
        char *blk = weights_at(c, bgl, rb, kt >> 2) + (kt & 3) * 2048 + lane * 16;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            __builtin_nontemporal_store(u32x4{pw[4 * f], pw[4 * f + 1], pw[4 * f + 2], pw[4 * f + 3]}, (u32x4 *)(blk + f * 1024));
            __builtin_nontemporal_store(u32x4{dw[4 * f], dw[4 * f + 1], dw[4 * f + 2], dw[4 * f + 3]}, (u32x4 *)(blk + 8192 + f * 1024));
        }
    };

    // One tile: three stages, one barrier; tile u is multiplied while tile u + 2 travels and the weights of u - 1 are formed.
    int st = 0;
    auto step = [&](int u, f32x16 &s_new, f32x16 &t_new, const f32x16 &s_old, const f32x16 &t_old) {
        // tile u has landed: behind its copies this wave issued 9 more, and 4 stores in either of the two steps since
        if (u < 3) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(17)" ::: "memory");
        lds_barrier();
        const TileCopy tc = plan_tile(u + 2, st == 0 ? 2 : st - 1);
        const uint32_t a_addr = smem_lds + st * kStageScores + ln * kRow1 + lh * 16;
        bf16x8 kf[LOZA_SCORE_DEPTH_576];
        uint32_t tmp, pw[8], dw[8];
        float w[6];
        LOZA_BWD_SCORES_K36_T32(s_new, t_new, kf, tmp, pw, dw, w, a_addr, xf, voff, s_old, t_old, lse2, dd, tc, wave, p.scale_log2, p.scale);
        if (u > 0) put(u - 1, pw, dw);
        st = st == 2 ? 0 : st + 1;
    };
    f32x16 s0, t0, s1, t1;
#pragma unroll
    for (int e = 0; e < 16; ++e) { s1[e] = 0.f; t1[e] = 0.f; }
    int u = 0;
    while (true) {
        step(u, s0, t0, s1, t1);
        if (++u == nt) break;
        step(u, s1, t1, s0, t0);
        if (++u == nt) { s0 = s1; t0 = t1; break; }
    }
    uint32_t pw[8], dw[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        float pe[2], de[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = 2 * x + h;
            pe[h] = __builtin_amdgcn_exp2f(__builtin_fmaf(s0[e], p.scale_log2, -lse2[e]));
            de[h] = p.scale * pe[h] * (t0[e] - dd[e]);
        }
        pw[x] = pack_bf16(pe[0], pe[1]);
        dw[x] = pack_bf16(de[0], de[1]);
    }
    put(nt - 1, pw, dw);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may still be on its way into LDS when the workgroup ends
}

// ---- the two products ------------------------------------------------------------------------------------
namespace {

// A 128 x 576 result, transposed: of a wave, columns 128 wave .. + 127 (four blocks of 32) for all four blocks of
// 32 rows or keys, and columns 512 .. 575 for block `wave`.
struct WideAcc {
    f32x16 a[4][4], rope[2];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y)
#pragma unroll
                for (int e = 0; e < 16; ++e) a[x][y][e] = 0.f;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int e = 0; e < 16; ++e) rope[x][e] = 0.f;
            asm volatile("" : "+v"(rope[x]));
        }
    }
};

// What the first matrix instructions of a tile need, read before the tile before it is through.
constexpr int kAhead = 3;
struct WideFrags {
    bf16x8 b[4], f[kAhead];
};

template <typename F>
__device__ __forceinline__ void each_copy(F &&f)
{
    f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{}); f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{}); f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{}); f(std::integral_constant<int, 8>{});
    f(std::integral_constant<int, 9>{}); f(std::integral_constant<int, 10>{}); f(std::integral_constant<int, 11>{});
}
// f(n) with n a constant (after unrolling)
template <typename F>
__device__ __forceinline__ void copy_const(F &&f, int n)
{
    each_copy([&](auto k) { if (decltype(k)::value == n) f(k); });
}

// acc += Y^T B over the 32 items of a tile: Y the streamed tile (padded rows of ROW bytes; y: address of this lane's first
// transposed read of column block 0, its second one `second` bytes further), B four blocks of 32 x 32 weights; b_of(block,
// ks): B fragment. copy(n): the n-th of 12 copy instructions, two products apart. Three quarters through, when all of
// this tile has been read, ready() waits for the next one and for the other waves, first(frags) reads its first operands, and
// plan() prepares the next copies: what a wave waits for (a barrier, LDS, scalar arithmetic) then has matrix work behind it.
// (The same cycles as with all of it between two tiles, while the copies are what a tile waits for.)
template <bool ROPE, int ROW, typename B, typename Copy, typename Ready, typename First, typename Plan>
__device__ __forceinline__ void wide_product(WideAcc &acc, WideFrags &fr, const char *y, const int second, const int wave, B &&b_of, Copy &&copy,
                                             Ready &&ready, First &&first, Plan &&plan)
{
    auto frag = [&](int m) {   // m = ks * 4 + column block
        const char *a = y + (m >> 2) * 16 * ROW + (m & 3) * 64;
        return read_tr_pair(a, a + second);
    };
    bf16x8 b[4], bn[4], f[8], rf[2], rb;
#pragma unroll
    for (int x = 0; x < 4; ++x) b[x] = fr.b[x];
#pragma unroll
    for (int m = 0; m < kAhead; ++m) f[m] = fr.f[m];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int n = m * 4 + x;
            acc.a[m & 3][x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m], m < 4 ? b[x] : bn[x], acc.a[m & 3][x], 0, 0, 0);
            if (x == 0 && m + kAhead < 8) f[m + kAhead] = frag(m + kAhead);
            if (m == 1) bn[x] = b_of(x, 1);
            if (ROPE && (m == 0 || m == 4) && (x == 1 || x == 2)) {
                const char *a = y + (m >> 2) * 16 * ROW + (16 + x - 1 - wave * 4) * 64;
                rf[x - 1] = read_tr_pair(a, a + second);
            }
            if (ROPE && (m == 0 || m == 4) && x == 3) rb = b_of(wave, m >> 2);
            if (n < 24 && (n & 1)) copy_const(copy, n >> 1);
            if (n == 23) ready();
            if (n == 24) first(fr);
            if (n == 28) plan();
            __builtin_amdgcn_sched_barrier(0);
        }
        if (ROPE && (m == 2 || m == 6)) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
                asm volatile("s_nop 1\n v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc.rope[x]) : "v"(rf[x]), "v"(rb));
        }
    }
}

}  // namespace

// dQ of 128 rows.
__global__ __launch_bounds__(256) void ssa_bwd_wide_dq_kernel(const BwdParams p, const WideChunk c)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, lh = lane >> 5;
    const int s16 = lane & 15, g16 = (lane >> 4) & 1;
    const int G = p.G;
    const int64_t S = p.S, R = S * G;
    const int n_t = c.t1 - c.t0, bgl = blockIdx.x / n_t, t = c.t1 - 1 - blockIdx.x % n_t;
    const int b = (c.bg0 + bgl) / p.Hkv, g = (c.bg0 + bgl) % p.Hkv;

    const RowTileKeys keys(p, R, (int64_t)t * 128, (int64_t)t * 128 + 128);
    int nA, wt0, nB;
    keys.pieces(5, nA, wt0, nB);
    const int nt = nA + nB;

    const uint32_t k_stride = (uint32_t)p.Hkv * (kDqk * 2);
    uint32_t voff[10];
#pragma unroll
    for (int x = 0; x < 10; ++x) voff[x] = chunk_offset<kRow1T, kDqk * 2>(x * 4 + wave, lane, key_item, k_stride, 0, 0);
    const char *k_base = (const char *)(p.k + ((int64_t)b * S * p.Hkv + g) * kDqk);
    // The weights lie [key][runs of 4 rows] and are read transposed. Chunk (half h, key) of a fragment of 1 KB goes to
    // place (h, key ^ 4 h): the 32 chunks that a read touches are then two in every 16 bytes of the 64 banks.
    const uint32_t woff = ((lane & 32) + ((lane & 31) ^ (lh * 4))) * 16;
    struct TileCopy { const char *src, *w; uint32_t max, dst, dstw; };
    int next_u = 0, next_stage = 0;                          // the tile to be copied next (the last one again behind the end)
    auto plan_next = [&]() {
        const int uu = next_u < nt ? next_u : nt - 1, kt = uu < nA ? uu : wt0 + (uu - nA);
        const int y0 = kt * 32, last = (int)S - 1 - y0 < 31 ? (int)S - 1 - y0 : 31;
        TileCopy tc;
        tc.src = k_base + (int64_t)y0 * k_stride;
        tc.w = weights_at(c, bgl, t * 4 + wave, kt >> 2) + 8192 + (kt & 3) * 2048;
        tc.max = last * k_stride + kDqk * 2 - 16;
        tc.dst = smem_lds + next_stage + wave * 1024;
        tc.dstw = smem_lds + next_stage + kOffB + wave * 2048;
        ++next_u;
        next_stage = next_stage == 2 * kStageProduct ? 0 : next_stage + kStageProduct;
        return tc;
    };
    auto copy_nth = [&](const TileCopy &tc, auto nc) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n < 2) copy_1k_once(tc.w, woff + n * 1024, tc.dstw + n * 1024);
        else if constexpr (n < 11) copy_1k_cut<(n - 2) * 4096>(tc.src, voff[n - 2], tc.max, tc.dst);
        else if (wave < kCopies1T - 36) copy_1k_cut<9 * 4096>(tc.src, voff[9], tc.max, tc.dst);
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const TileCopy tc = plan_next();
        each_copy([&](auto n) { copy_nth(tc, n); });
    }

    WideAcc acc;
    acc.clear();
    const int y_lane = (lh * 8 + (s16 >> 2)) * kRow1T + (g16 * 16 + (s16 & 3) * 4) * 2 + wave * 256;
    const int w_h = s16 & 1, w_key = lh * 8 + (s16 >> 2);
    const int w_at = kOffB + g16 * 1024 + (w_h * 32 + w_key) * 16 + ((s16 >> 1) & 1) * 8;
    const int w_lo = w_at + w_h * 64, w_hi = w_at + 64 - w_h * 64;   // keys .. + 3; + 4 .. + 7
    auto weights = [&](const char *tile, int x, int ks) { return read_tr_pair(tile + w_lo + x * 2048 + ks * 256, tile + w_hi + x * 2048 + ks * 256); };
    int st = 0;
    WideFrags fr;
    auto ready = [&]() {
        asm volatile("s_waitcnt vmcnt(11)" ::: "memory");   // the next tile has landed; the 11 (or 12) copies behind it may be on their way
        lds_barrier();
        st = st == 2 * kStageProduct ? 0 : st + kStageProduct;
    };
    auto first = [&](WideFrags &f) {
        const char *tile = smem + st;
#pragma unroll
        for (int x = 0; x < 4; ++x) f.b[x] = weights(tile, x, 0);
#pragma unroll
        for (int m = 0; m < kAhead; ++m) f.f[m] = read_tr_pair(tile + y_lane + m * 64, tile + y_lane + m * 64 + 4 * kRow1T);
    };
    asm volatile("s_waitcnt vmcnt(11)" ::: "memory");
    lds_barrier();
    first(fr);
    TileCopy tc = plan_next();
    for (int u = 0; u < nt; ++u) {
        const char *tile = smem + st;
        const TileCopy now = tc;
        wide_product<true, kRow1T>(acc, fr, tile + y_lane, 4 * kRow1T, wave, [&](int x, int ks) { return weights(tile, x, ks); },
            [&](auto n) { copy_nth(now, n); }, ready, first, [&]() { tc = plan_next(); });
    }
    asm volatile("s_waitcnt vmcnt(0)\n s_nop 7\n s_nop 7\n s_nop 7" : "+v"(acc.rope[0]), "+v"(acc.rope[1]) :: "memory");

    // Through LDS, so that rows leave in whole lines: a lane holds four columns of a row, and 8 bytes of 32 rows an
    // instruction keep the address unit busy for longer than the products of eight tiles take.
    lds_barrier();
    auto put = [&](const f32x16 &v, int x, int col) {        // block x of 32 rows, 32 columns from col on
        char *at = smem + (x * 32 + ln) * kRowOut + (col + 4 * lh) * 2;
#pragma unroll
        for (int qd = 0; qd < 4; ++qd)
            *(u32x2 *)(at + qd * 16) = u32x2{pack_bf16(v[4 * qd], v[4 * qd + 1]), pack_bf16(v[4 * qd + 2], v[4 * qd + 3])};
    };
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int a = 0; a < 4; ++a) put(acc.a[a][x], x, wave * 128 + a * 32);
    put(acc.rope[0], wave, 512);
    put(acc.rope[1], wave, 544);
    lds_barrier();
#pragma unroll 6
    for (int n = 0; n < 36; ++n) {                           // 32 rows of 72 chunks of 16 bytes a wave
        const int q = n * 64 + lane, row = wave * 32 + q / 72, ch = q % 72;
        const int64_t r = (int64_t)t * 128 + row;
        const u32x4 v = *(const u32x4 *)(smem + row * kRowOut + ch * 16);
        if (r < R) {
            const int64_t i = row_position(r, G);
            *(u32x4 *)(p.dq + (((int64_t)b * S + i) * p.Hq + (int64_t)g * G + (r - i * G)) * kDqk + ch * 8) = v;
        }
    }
}

// Partial dK (with dV) of 128 keys over a segment of the chunk's rows.
__global__ __launch_bounds__(256) void ssa_bwd_wide_dk_kernel(const BwdParams p, const WideChunk c)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lh = lane >> 5;
    const int s16 = lane & 15, g16 = (lane >> 4) & 1;
    const int G = p.G;
    const int64_t S = p.S, R = S * G;
    // Workgroups go to the eight XCDs round-robin: the key groups of a segment, which stream the same rows, to one of
    // them and one after the other, so that one fetch into its L2 serves all.
    const int xcd = blockIdx.x % 8, j = blockIdx.x / 8 % c.max_groups, seg = blockIdx.x / 8 / c.max_groups * 8 + xcd;
    if (seg >= c.nbg * c.n_seg) return;
    const int bgl = seg / c.n_seg, b = (c.bg0 + bgl) / p.Hkv, g = (c.bg0 + bgl) % p.Hkv;
    int ta = c.t0 + seg % c.n_seg * c.seg_tiles, tb = ta + c.seg_tiles < c.t1 ? ta + c.seg_tiles : c.t1;
    if (ta >= tb) return;
    int gA, wg0, gB;
    RowTileKeys(p, R, (int64_t)ta * 128, (int64_t)tb * 128).pieces(7, gA, wg0, gB);
    if (j >= gA + gB) return;
    const int kg = j < gA ? j : wg0 + (j - gA);
    // row tiles of the segment that see a key of the group
    group_rows(p, kg, ta, tb, ta, tb);
    const int rb0 = ta * 4, rb_end = tb * 4 < (int)((R + 31) / 32) ? tb * 4 : (int)((R + 31) / 32), n_rb = rb_end - rb0;

    int g_shift = 5;
    if (G < 32) g_shift = __builtin_ctz((unsigned)G);
    const int g_log2 = (G & (G - 1)) == 0 ? __builtin_ctz((unsigned)G) : -1;
    uint32_t voff1[10], voff2[9];
#pragma unroll
    for (int x = 0; x < 10; ++x) voff1[x] = chunk_offset<kRow1T, kDqk * 2>(x * 4 + wave, lane, row_item, (uint32_t)p.Hq * (kDqk * 2), kDqk * 2, g_shift);
#pragma unroll
    for (int x = 0; x < 9; ++x) voff2[x] = chunk_offset<kRow2T, kDv * 2>(x * 4 + wave, lane, row_item, (uint32_t)p.Hq * (kDv * 2), kDv * 2, g_shift);
    const int64_t row_base = (int64_t)b * S * p.Hq + (int64_t)g * G;
    // half-step 2 n: q rows of row block n and dS; 2 n + 1: dO rows and p
    struct TileCopy { const char *src, *w; uint32_t max, dst, dstw; };
    const int ragged = (int)R - (rb_end - 1) * 32 - 1;       // last row of the last block, within it (31 and more: whole)
    auto max_of = [&](int last, uint32_t width) { return row_item(last < 31 ? last : 31, (uint32_t)p.Hq * width, width, g_shift) + width - 16; };
    const uint32_t full1 = max_of(31, kDqk * 2), full2 = max_of(31, kDv * 2), cut1 = max_of(ragged, kDqk * 2), cut2 = max_of(ragged, kDv * 2);
    int next_n = 0, next_stage = 0;                          // the row block to be copied next (the last one again behind the end)
    const int i0 = (int)row_position((int64_t)rb0 * 32, G);
    int next_h = rb0 * 32 - i0 * G;                          // its first row's head within the group
    const char *next_q = (const char *)(p.q + (row_base + (int64_t)i0 * p.Hq + next_h) * kDqk), *next_d = (const char *)(p.dout + (row_base + (int64_t)i0 * p.Hq + next_h) * kDv);
    const char *next_w = weights_at(c, bgl, rb0, kg);
    const int64_t w_step = (int64_t)c.slots * kBlockBytes;
    auto plan_next = [&](bool second) {
        TileCopy tc;
        tc.src = second ? next_d : next_q;
        tc.w = second ? next_w : next_w + 8192;
        tc.max = next_n == n_rb - 1 ? (second ? cut2 : cut1) : (second ? full2 : full1);
        tc.dst = smem_lds + next_stage + wave * 1024;
        tc.dstw = smem_lds + next_stage + kOffB + wave * 2048;
        next_stage = next_stage == 2 * kStageProduct ? 0 : next_stage + kStageProduct;
        if (second && next_n < n_rb - 1) {
            ++next_n;
            int rows = 32;                                   // tensor rows to the next block's first
            if (G < 32) rows = (32 >> g_shift) * p.Hq;
            else if ((next_h += 32) == G) { next_h = 0; rows += p.Hq - G; }
            next_q += (int64_t)rows * (kDqk * 2);
            next_d += (int64_t)rows * (kDv * 2);
            next_w += w_step;
        }
        return tc;
    };
    const uint32_t woff = lane * 16 + wave * 2048;
    auto copy_first = [&](const TileCopy &tc, auto nc) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n < 2) copy_1k_once(tc.w, woff + n * 1024, tc.dstw + n * 1024);
        else if constexpr (n < 11) copy_1k_cut<(n - 2) * 4096>(tc.src, voff1[n - 2], tc.max, tc.dst);
        else if (wave < kCopies1T - 36) copy_1k_cut<9 * 4096>(tc.src, voff1[9], tc.max, tc.dst);
    };
    auto copy_second = [&](const TileCopy &tc, auto nc) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n < 2) copy_1k_once(tc.w, woff + n * 1024, tc.dstw + n * 1024);
        else if constexpr (n < 10) copy_1k_cut<(n - 2) * 4096>(tc.src, voff2[n - 2], tc.max, tc.dst);
        else if constexpr (n == 10) { if (wave < kCopies2T - 32) copy_1k_cut<8 * 4096>(tc.src, voff2[8], tc.max, tc.dst); }
    };
    {
        const TileCopy a = plan_next(false), d = plan_next(true);
        each_copy([&](auto n) { copy_first(a, n); });
        each_copy([&](auto n) { copy_second(d, n); });
    }

    WideAcc acc;
    acc.clear();
    // (a lane's weights are those of rows 4 h .. + 3 and 8 + 4 h .. + 3 of a step of 16: the rows are read in that order too)
    const int y_col = (g16 * 16 + (s16 & 3) * 4) * 2 + wave * 256, y_row = lh * 4 + (s16 >> 2), w_lane = kOffB + lane * 16;
    const int y1 = y_row * kRow1T + y_col, y2 = y_row * kRow2T + y_col;
    int st = 0;
    WideFrags fr;
    auto next_tile = [&]() { st = st == 2 * kStageProduct ? 0 : st + kStageProduct; };
    auto first = [&](WideFrags &f, int y, int second) {
        const char *tile = smem + st;
#pragma unroll
        for (int x = 0; x < 4; ++x) f.b[x] = *(const bf16x8 *)(tile + w_lane + x * 2048);
#pragma unroll
        for (int m = 0; m < kAhead; ++m) f.f[m] = read_tr_pair(tile + y + m * 64, tile + y + m * 64 + second);
    };
    asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
    lds_barrier();
    first(fr, y1, 8 * kRow1T);
    TileCopy tc = plan_next(false);
    for (int n = 0; n < n_rb; ++n) {
        {
            const char *tile = smem + st;
            const TileCopy now = tc;
            wide_product<true, kRow1T>(acc, fr, tile + y1, 8 * kRow1T, wave, [&](int x, int ks) { return *(const bf16x8 *)(tile + w_lane + x * 2048 + ks * 1024); },
                [&](auto m) { copy_first(now, m); },
                [&]() { asm volatile("s_waitcnt vmcnt(11)" ::: "memory"); lds_barrier(); next_tile(); },   // behind the next half-step's copies: this one's 11 (or 12)
                [&](WideFrags &f) { first(f, y2, 8 * kRow2T); }, [&]() { tc = plan_next(true); });
        }
        {
            const char *tile = smem + st;
            const TileCopy now = tc;
            wide_product<false, kRow2T>(acc, fr, tile + y2, 8 * kRow2T, wave, [&](int x, int ks) { return *(const bf16x8 *)(tile + w_lane + x * 2048 + ks * 1024); },
                [&](auto m) { copy_second(now, m); },
                [&]() { asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); lds_barrier(); next_tile(); },
                [&](WideFrags &f) { first(f, y1, 8 * kRow1T); }, [&]() { tc = plan_next(false); });
        }
    }
    asm volatile("s_waitcnt vmcnt(0)\n s_nop 7\n s_nop 7\n s_nop 7" : "+v"(acc.rope[0]), "+v"(acc.rope[1]) :: "memory");

    // partial sums in the order of the registers: [column block][key block][run of four][lane]
    float4 *out = (float4 *)c.part + ((int64_t)seg * c.max_groups + j) * (128 * kDqk / 4) + lane;
    auto store = [&](const f32x16 &v, int x, int db) {
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) out[((db * 4 + x) * 4 + qd) * 64] = float4{v[4 * qd], v[4 * qd + 1], v[4 * qd + 2], v[4 * qd + 3]};
    };
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int a = 0; a < 4; ++a) store(acc.a[a][x], x, wave * 4 + a);
    store(acc.rope[0], wave, 16);
    store(acc.rope[1], wave, 17);
}

// The chunk's partial sums of a key group, in the order of the segments, onto those of the chunks before; rounded
// and written out where no later chunk sees the group. Sums that go on are those of sink groups and of
// groups that rows on both sides of the chunk's end see: no two of them have the same place. But one that begins in
// this chunk can have the place of one that ends in it, so sums are read from one buffer and written to another, which the next
// chunk reads (one buffer where every group has a place). (A group that goes on beyond two ends is seen by the rows between them, and so is written again.) A workgroup
// is a 72nd of a group.
__global__ __launch_bounds__(256) void ssa_bwd_wide_reduce_kernel(const BwdParams p, const WideChunk c)
{
    const int G = p.G;
    const int64_t R = p.S * G;
    int gA, wg0, gB;
    RowTileKeys(p, R, (int64_t)c.t0 * 128, (int64_t)c.t1 * 128).pieces(7, gA, wg0, gB);
    const int n_g = gA + gB, at = blockIdx.x % 72 * 256 + threadIdx.x, x = blockIdx.x / 72 % n_g, bgl = blockIdx.x / 72 / n_g;
    if (bgl >= c.nbg) return;
    const int kg = x < gA ? x : wg0 + (x - gA);
    float4 s = {0.f, 0.f, 0.f, 0.f};
    const int64_t sum_at = (int64_t)(c.acc_in == c.acc_out ? kg : group_slot(c, kg)) * (128 * kDqk / 4) + at;
    if (c.t0 > kg * G) s = ((const float4 *)c.acc_in)[sum_at];
    // The segments with rows that see the group follow each other. (Eight loads in flight: one after the other, the many
    // segments of a sink group waited for memory each; 106 us a chunk of 455 partial sums while all segments were asked.)
    int see0, see1;
    group_rows(p, kg, c.t0, c.t1, see0, see1);
    const int last = (see1 - 1 - c.t0) / c.seg_tiles;
    for (int s0 = (see0 - c.t0) / c.seg_tiles; s0 <= last; s0 += 8) {
        float4 v[8];
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const int seg = s0 + h < last ? s0 + h : last, ta = c.t0 + seg * c.seg_tiles, tb = ta + c.seg_tiles < c.t1 ? ta + c.seg_tiles : c.t1;
            int sA, sw0, sB;
            RowTileKeys(p, R, (int64_t)ta * 128, (int64_t)tb * 128).pieces(7, sA, sw0, sB);
            const int j = kg < sA ? kg : sA + kg - sw0;
            v[h] = ((const float4 *)c.part)[((int64_t)(bgl * c.n_seg + seg) * c.max_groups + j) * (128 * kDqk / 4) + at];
        }
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            if (s0 + h > last) break;
            s.x += v[h].x; s.y += v[h].y; s.z += v[h].z; s.w += v[h].w;
        }
    }
    bool later = c.t1 < (int)((R + 127) / 128);
    if (later && kg * 128 >= p.n_sink) {
        const int64_t i_w = ((int64_t)(kg * 128 + 127) / p.block + p.window) * p.block - 1;
        later = (int64_t)c.t1 * 128 <= i_w * G + G - 1;
    }
    if (later) {
        ((float4 *)c.acc_out)[sum_at] = s;
        return;
    }
    const int lane = at & 63, blk = at >> 6;                 // [column block][key block][run of four]
    const int64_t key = (int64_t)kg * 128 + (blk >> 2 & 3) * 32 + (lane & 31);
    if (key >= p.S) return;
    const int b = (c.bg0 + bgl) / p.Hkv, g = (c.bg0 + bgl) % p.Hkv;
    *(u32x2 *)(p.dk + (((int64_t)b * p.S + key) * p.Hkv + g) * kDqk + (blk >> 4) * 32 + 8 * (blk & 3) + 4 * (lane >> 5)) =
        u32x2{pack_bf16(s.x, s.y), pack_bf16(s.z, s.w)};
}

hipError_t launch_bwd_wide(const BwdParams &p, const WidePlan &w, hipStream_t stream)
{
    hipError_t e;
    if ((e = allow_lds<ssa_bwd_wide_scores_kernel>(kLdsScores)) != hipSuccess) return e;
    if ((e = allow_lds<ssa_bwd_wide_dq_kernel>(kLdsDq)) != hipSuccess) return e;
    if ((e = allow_lds<ssa_bwd_wide_dk_kernel>(kLdsProduct)) != hipSuccess) return e;
    const int BH = p.B * p.Hkv;
    WideChunk c = w.chunk;   // (the first chunk of a (batch, key head) reads no sums)
    for (int bg = 0; bg < BH; bg += w.chunk_bgs) {
        for (int t = 0; t < w.row_tiles; t += w.chunk_tiles) {
            c.bg0 = bg;
            c.nbg = BH - bg < w.chunk_bgs ? BH - bg : w.chunk_bgs;
            c.t0 = t;
            c.t1 = w.row_tiles - t < w.chunk_tiles ? w.row_tiles : t + w.chunk_tiles;
            c.n_seg = (c.t1 - c.t0 + c.seg_tiles - 1) / c.seg_tiles;
            const unsigned tiles = (unsigned)((c.t1 - c.t0) * c.nbg), segs = (unsigned)(c.n_seg * c.nbg + 7) / 8 * 8;
            hipLaunchKernelGGL(ssa_bwd_wide_scores_kernel, dim3(tiles), dim3(256), kLdsScores, stream, p, c);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(ssa_bwd_wide_dk_kernel, dim3(segs * c.max_groups), dim3(256), kLdsProduct, stream, p, c);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(ssa_bwd_wide_dq_kernel, dim3(tiles), dim3(256), kLdsDq, stream, p, c);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            // key groups that the chunk's rows see
            const int64_t r1 = (int64_t)c.t1 * 128 < p.S * p.G ? (int64_t)c.t1 * 128 : p.S * p.G;
            const int i_min = (int)((int64_t)c.t0 * 128 / p.G), i_max = (int)((r1 - 1) / p.G);
            const int sinks = (int)(((p.n_sink < i_max + 1 ? p.n_sink : i_max + 1) + 127) / 128), w0 = window_begin_of(i_min, p.window, p.block) / 128;
            const unsigned n_g = (unsigned)(w0 <= sinks ? i_max / 128 + 1 : sinks + i_max / 128 - w0 + 1);
            hipLaunchKernelGGL(ssa_bwd_wide_reduce_kernel, dim3(72 * n_g * c.nbg), dim3(256), 0, stream, p, c);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            float *sums = c.acc_in;
            c.acc_in = c.acc_out;
            c.acc_out = sums;
        }
    }
    return hipSuccess;
}

}  // namespace loza
