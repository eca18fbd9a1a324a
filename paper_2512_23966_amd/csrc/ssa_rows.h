// Sixteen query rows of one key/value head against their live keys: the pass that the kernels for few query rows
// are made of (ssa_rows.hip).
//
// The tile kernel of ssa_bf16.hip gives a workgroup 64 (decode) or 128 query rows and lets its four
// waves share every key tile, which is right where rows are plenty. With few rows it leaves the chip
// idle (4 new tokens for 16 sequences are 32 such tiles on 256 compute units) or, in a decode, has to
// cut the keys so finely that the fp32 partial results weigh as much as the keys themselves. Here a
// workgroup owns 16 query rows (position, head) of one key/value head and its four waves share the
// KEYS: wave w of split s takes every (4 n_splits)-th tile of 16 live keys, keeps its own softmax state and its
// own output accumulators (all d_v columns of the 16 rows), and the four partial results meet in LDS
// once, at the end. Consequences:
//   * no barrier and no hand-over inside the loop: the probabilities of a tile are already where the
//     next matrix instruction wants them. S^T[16 keys][16 rows] = K Q^T leaves lane (j, n) with row n's
//     scores of keys 4j .. 4j + 3, and the B operand of O^T += V^T P^T wants from lane (j, n) eight
//     values of row n along the contraction, whose order is free: slots 0..3 are the four keys' weights
//     rounded to bf16, slots 4..7 what that rounding lost (again bf16), and the A operand carries the
//     four keys' values twice. One 16x16x32 instruction thus accumulates 16 keys with weights good to
//     2^-17, at the price of one-term weights: no row has to be computed again because it is large or
//     has few live keys. A decode takes what two terms leave as a third, in an instruction of its own: three
//     bf16 terms hold all 24 bits of an fp32 weight (43 sequences of 1,024 live keys, wide shape: 33.0 us with
//     it, 30.3 without; 8,192 live keys of one sequence 18.7 and 17.8; d = 128, 16 sequences: no difference).
//   * each key row is read from LDS once for the scores and once (transposing) for the values per 16
//     rows (16 keys of the wide shape: 18 KB at 104 B/clk, 16 KB at 64 B/clk and the incoming 18 KB: about 580 cycles
//     per tile and compute unit; the LDS is busy 20 % of the time). With one wave a SIMD what bounds the loop is latency
//     and issue of a wave's chain of scores, softmax and values (matrix cores busy 28 %, vector units 25 %).
//   * (M = 32 rows a workgroup, two blocks of 16 that share every read, where width 128 has more than a round of groups)
//   * workgroups that walk the same keys for other rows are placed on the same XCD, whose L2 then serves
//     all but the first of them.
// Tiles travel global -> LDS with global_load_lds_dwordx4 into a ring of NST stages per wave; the copy of
// tile t + NST - 1 is issued whole before the scores of tile t (its instructions between the LDS reads of the
// score phase serialised those). The softmax reference is a row's maximum over its first tile and moves only when
// exceeded by 2^8. A stage holds 16 unpadded rows; the 16-byte
// chunks of a row are permuted within groups of eight (chunk c of row r sits in slot c ^ (r & 7)), which
// costs nothing (the copy fetches whatever chunk belongs into its slot) and makes both kinds of reads
// free of bank conflicts.
#ifndef LOZA_SSA_ROWS_H
#define LOZA_SSA_ROWS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssa_device.h"
#include "ssa_direct.h"
#include "ssa_kernels.h"

namespace loza {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// One global -> LDS copy instruction (1 KB), unknown to the compiler's wait counters: the loop waits
// with explicit counts. NT: the rows are read by this workgroup only (non-temporal hint).
template <bool NT>
__device__ __forceinline__ void copy_1k(const char *base, uint32_t off, uint32_t lds_addr)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1 nt"
                     :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1"
                     :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void wait_copies()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// max over the four lanes (lane & 15) + 16 j, in every one of them
__device__ __forceinline__ float max_over_groups(float x)
{
    x = max_with_other_half(x);
    // v_permlane16_swap exchanges odd 16-lane rows of its first operand with even rows of the second
    uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
    asm volatile("" : "+v"(b));
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    uint32_t r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1));
    return fmaxf(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));
}

}  // namespace

template <int DQK, int DV, bool ALIAS>
struct RowsCfg {
    static constexpr int N = 16;                       // keys per tile
    static constexpr int NW = 4;                       // waves
    static constexpr int CK = DQK / 8, CV = DV / 8;    // 16-byte chunks per row
    static_assert(CK % 8 == 0 && CV % 8 == 0, "chunks are permuted in groups of eight");
    static constexpr int KBYTES = N * CK * 16, VBYTES = ALIAS ? 0 : N * CV * 16;
    static constexpr int KI = KBYTES / 1024, VI = VBYTES / 1024, NI = KI + VI;   // copy instructions per tile
    static_assert(KI * 1024 == KBYTES && VI * 1024 == VBYTES, "whole copy instructions");
    static constexpr int STAGE = KBYTES + VBYTES;
    // wide rows: two stages of 18 KB per wave fill the LDS; narrow rows: four stages
    static constexpr int NST = STAGE > 16384 ? 2 : 4;
    static constexpr int OROW = DV * 4 + 16;           // LDS bytes per row of a wave's partial output
    static constexpr int REGION = NST * STAGE > N * OROW ? NST * STAGE : N * OROW;
    static constexpr int OFF_ML = NW * REGION;         // float[NW][16][2]: reference maximum, sum
    static constexpr int OFF_ODD = OFF_ML + NW * 16 * 8;   // uint32_t: finished rows that hold a NaN or an infinity
    static constexpr int LDS_BYTES = OFF_ODD + 16;
    static_assert(LDS_BYTES + 4096 <= 160 * 1024, "does not fit the 160 KB LDS");   // (and decode_row_direct's)
};

// One pass: rows M rt .. M rt + M - 1 (M = 16 MB) of (batch b, key head g), tiles `split` of n_splits. EXACT: three-term weights
// (decode). NT: the key rows are read by this workgroup only. All 256 threads call it together; the LDS it uses
// (RowsCfg::LDS_BYTES) must not be in use when it starts.
template <int DQK, int DV, bool ALIAS, bool NT, bool EXACT, int MB>
__device__ __forceinline__ void ssa_rows_pass(const FwdParams &p, char *smem, const int b, const int g, const int rt, const int split, const int n_splits)
{
    using C = RowsCfg<DQK, DV, ALIAS>;
    constexpr int N = C::N, NST = C::NST, AHEAD = NST - 1, M = 16 * MB;
    static_assert(MB == 1 || !EXACT, "decodes take 16 rows");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n16 = lane & 15, j4 = lane >> 4;
    const int G = p.G;
    const bool cached = p.seqlens != nullptr;      // queries are the last q_len positions of a cache
    const int64_t L = cached ? ((int64_t)p.seqlens[b] < p.S ? (int64_t)p.seqlens[b] : p.S) : p.S;
    const int64_t Sq = cached ? (int64_t)p.q_len : p.S;
    const int64_t pos0 = L - Sq;
    const int64_t R = Sq * G, r0 = (int64_t)rt * M;
    const int n_sink = p.n_sink, window = p.window, block = p.block;
    const int i_min = (int)(pos0 + row_position(r0, G));
    const int i_max = (int)(pos0 + row_position((r0 + M - 1 < R) ? r0 + M - 1 : R - 1, G));

    // ---- this wave's live key tiles: sink tiles [0, nA), then window tiles [wt0, wt0 + nB), dealt out ---
    const int sink_end = i_max < 0 ? 0 : (n_sink < i_max + 1 ? n_sink : i_max + 1);
    const int win_begin = window_begin_of(i_min < 0 ? 0 : i_min, window, block);
    const int w_lo_max = window_begin_of(i_max < 0 ? 0 : i_max, window, block);
    int nA = (sink_end + N - 1) / N;
    const int wt0 = win_begin / N, wt1 = i_max / N;
    int nB;
    if (wt0 <= nA) { nA = wt1 + 1; nB = 0; } else { nB = wt1 - wt0 + 1; }
    if (i_max < 0) { nA = 0; nB = 0; }
    const int first = split * C::NW + wave, stride = n_splits * C::NW;
    const int nt = nA + nB > first ? (nA + nB - first + stride - 1) / stride : 0;
    auto key_tile = [&](int t) {
        const int tt = first + t * stride;
        return tt < nA ? tt : wt0 + (tt - nA);
    };

    // ---- copies ----------------------------------------------------------------------------------------
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const uint32_t ring = smem_lds + wave * C::REGION;
    const uint32_t k_stride = (uint32_t)p.Hkv * DQK * 2, v_stride = (uint32_t)p.Hkv * DV * 2;
    // slot i * 64 + lane of a sub-tile holds chunk slot % cpr (permuted) of row slot / cpr
    auto offset_of = [&](int i, int cpr, uint32_t row_stride, int row_max) -> uint32_t {
        const int slot = i * 64 + lane, row = slot / cpr, c = slot - row * cpr;
        const int chunk = (c & ~7) | ((c ^ row) & 7);
        return (uint32_t)(row < row_max ? row : row_max) * row_stride + (uint32_t)chunk * 16u;
    };
    uint32_t off[C::NI];
#pragma unroll
    for (int i = 0; i < C::NI; ++i)
        off[i] = i < C::KI ? offset_of(i, C::CK, k_stride, N - 1) : offset_of(i - C::KI, C::CV, v_stride, N - 1);
    const bool paged = p.block_table != nullptr;
    const int64_t seq_row0 = paged ? 0 : (int64_t)b * p.S;
    const char *kbase = (const char *)p.k + (seq_row0 * p.Hkv + g) * (int64_t)DQK * 2;
    const char *vbase = (const char *)p.v + (seq_row0 * p.Hkv + g) * (int64_t)DV * 2;
    // (a scalar load the compiler knows about: it waits before the first use; entries past the row read 0)
    const i32x4 table_rsrc = paged ? table_row_resource(p.block_table + (int64_t)b * p.max_pages, p.max_pages) : i32x4{0, 0, 0, 0};
    auto page_of = [&](int t) -> int32_t {
        if (!paged) return 0;
        const int64_t j0 = (int64_t)key_tile(t) * N;
        return llvm_amdgcn_s_buffer_load_i32(table_rsrc, (int32_t)((uint32_t)(j0 >> p.page_shift) * 4u), 0);
    };
    struct TileCopy {
        const char *k, *v;
        uint32_t dst;
        int rows;          // rows of the tile that exist, minus one (at most N - 1)
    };
    auto plan = [&](int t, int stage, int32_t pid) {
        const int64_t j0 = (int64_t)key_tile(t) * N;
        int64_t row = j0;
        if (paged) {
            pid = pid < 0 ? 0 : (pid < p.num_pages ? pid : p.num_pages - 1);   // a bad entry stays in bounds
            row = ((int64_t)pid << p.page_shift) + (j0 & ((1 << p.page_shift) - 1));
        }
        TileCopy tc;
        tc.k = kbase + row * (int64_t)k_stride;
        tc.v = vbase + row * (int64_t)v_stride;
        tc.dst = ring + stage * C::STAGE;
        const int left = (int)(L - 1 - j0);
        tc.rows = left < N - 1 ? left : N - 1;
        return tc;
    };
    // copy instruction i of a tile whose rows all exist
    auto copy_nth = [&](const TileCopy &tc, int i) { copy_1k<NT>(i < C::KI ? tc.k : tc.v, off[i], tc.dst + i * 1024); };
    // the tile that holds the sequence end: rows past it fetch the last valid row instead (they are dead
    // and only have to be finite)
    auto copy_ragged = [&](const TileCopy &tc) {
#pragma unroll
        for (int i = 0; i < C::NI; ++i) {
            const uint32_t o = i < C::KI ? offset_of(i, C::CK, k_stride, tc.rows) : offset_of(i - C::KI, C::CV, v_stride, tc.rows);
            copy_1k<NT>(i < C::KI ? tc.k : tc.v, o, tc.dst + i * 1024);
        }
    };
    auto copy_tile = [&](const TileCopy &tc) {
        if (tc.rows < N - 1) { copy_ragged(tc); return; }
#pragma unroll
        for (int i = 0; i < C::NI; ++i) copy_nth(tc, i);
    };

#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (a < nt) copy_tile(plan(a, a, page_of(a)));

    // ---- the queries: matrix-core B operands, row n16 of each block of 16 ------------------------------
    constexpr int KS = DQK / 32;
    bf16x8 qf[MB][KS];
    int i_row[MB], w_lo_row[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int64_t row = r0 + mb * 16 + n16, rc = row < R ? row : R - 1;
        const int64_t qi = row_position(rc, G);
        const int hh = (int)(rc - qi * G);
        i_row[mb] = (int)(pos0 + qi);
        w_lo_row[mb] = window_begin_of(i_row[mb] < 0 ? 0 : i_row[mb], window, block);
        const uint16_t *qp = p.q + (((int64_t)b * Sq + qi) * p.Hq + (int64_t)g * G + hh) * DQK + j4 * 8;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[mb][kk] = *(const bf16x8 *)(qp + kk * 32);
    }
    // (waited for here, with a wait the compiler sees: left to its own bookkeeping it would wait for the
    // queries inside the loop, with counts that also drain the tile copies it does not know about)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[mb][kk]));

    constexpr int CB = DV / 16;   // column blocks
    f32x4 o[MB][CB];
    float m_ref[MB], l_run[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        m_ref[mb] = LOZA_NEG_INF;
        l_run[mb] = 0.f;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) o[mb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // per-lane LDS offsets of the reads, within a stage
    const uint32_t krd[2] = {(uint32_t)(n16 * C::CK * 16 + ((j4 ^ (n16 & 7)) * 16)),
                             (uint32_t)(n16 * C::CK * 16 + (((4 + j4) ^ (n16 & 7)) * 16))};
    uint32_t vrd[4];
    {
        const int vr = j4 * 4 + (n16 >> 2);                       // row this lane addresses in a transposing read
        const int row_bytes = ALIAS ? C::CK * 16 : C::CV * 16;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            vrd[c] = (uint32_t)((ALIAS ? 0 : C::KBYTES) + vr * row_bytes + (((c * 2 + ((n16 & 3) >> 1)) ^ (vr & 7)) * 16) + (n16 & 1) * 8);
    }

    // ---- the tile loop: every wave on its own ------------------------------------------------------------
    int st = 0;
    int32_t pid = AHEAD < nt ? page_of(AHEAD) : 0;
    for (int t = 0; t < nt; ++t) {
        // tile t has landed when at most the copies of the tiles after it are outstanding
        if (t + AHEAD <= nt) wait_copies<(AHEAD - 1) * C::NI>();
        else wait_copies<0>();
        const int st_l = st == 0 ? NST - 1 : st - 1;              // the stage tile t - 1 has left
        const char *tile = smem + wave * C::REGION + st * C::STAGE;
        if (t + AHEAD < nt) copy_tile(plan(t + AHEAD, st_l, pid));
        pid = t + 1 + AHEAD < nt ? page_of(t + 1 + AHEAD) : 0;

        // scores: S^T[16 keys][16 rows], on two accumulators
        f32x4 s2[MB][2];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) s2[mb][0] = s2[mb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const bf16x8 a = *(const bf16x8 *)(tile + krd[kk & 1] + (kk >> 1) * 128);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) s2[mb][kk & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[mb][kk], s2[mb][kk & 1], 0, 0, 0);
        }
        const int j0 = key_tile(t) * N;
        const bool interior = (j0 + N - 1 <= i_min) && ((j0 + N - 1 < n_sink) || (j0 >= w_lo_max));
        bf16x8 pb[MB];
        u32x4 w3 = {0, 0, 0, 0};
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            f32x4 s = s2[mb][0] + s2[mb][1];
            if (!interior) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = j0 + 4 * j4 + e;
                    const bool ok = (j <= i_row[mb]) & ((j < n_sink) | (j >= w_lo_row[mb]));
                    s[e] = ok ? s[e] : LOZA_NEG_INF;
                }
            }
            float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * p.scale_log2;   // scale > 0
            // the reference moves when some row exceeds it by 2^8 (or has none yet): then every row of the
            // block takes its running maximum
            if (__any(mx > m_ref[mb] + p.lazy_log2)) {
                mx = max_over_groups(mx);
                const float m_new = fmaxf(m_ref[mb], mx);
                const float a = m_new == LOZA_NEG_INF ? 1.0f : __builtin_amdgcn_exp2f(m_ref[mb] - m_new);
                m_ref[mb] = m_new;
                l_run[mb] *= a;
                if (t > 0) {   // (not behind the first tile, whose accumulators are 0: 2,000 cycles; one sequence of window 8192 18.6 -> 17.4 us)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    // (the accumulators live in the AGPR half of the register file; pinned there on both
                    // sides of the multiply, four at a time pass through VGPRs, here and nowhere else)
                    f32x4 x = o[mb][cb];
                    asm volatile("" : "+a"(x));
                    x *= a;
                    asm volatile("" : "+a"(x));
                    o[mb][cb] = x;
                }
                }
            }
            const float m_use = m_ref[mb] == LOZA_NEG_INF ? 0.f : m_ref[mb];   // a row with no live key so far
            float e4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) e4[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], p.scale_log2, -m_use));
            l_run[mb] += (e4[0] + e4[1]) + (e4[2] + e4[3]);
            u32x4 w;
            w[0] = pack_bf16(e4[0], e4[1]);
            w[1] = pack_bf16(e4[2], e4[3]);
            auto lost = [](float x, uint32_t pair, int half) {        // what rounding x to that half of the pair lost
                return x - __builtin_bit_cast(float, half ? pair & 0xffff0000u : pair << 16);
            };
            float r4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r4[e] = lost(e4[e], w[e >> 1], e & 1);
            w[2] = pack_bf16(r4[0], r4[1]);
            w[3] = pack_bf16(r4[2], r4[3]);
            pb[mb] = __builtin_bit_cast(bf16x8, w);
            if constexpr (EXACT) {
                w3[0] = pack_bf16(lost(r4[0], w[2], 0), lost(r4[1], w[2], 1));
                w3[1] = pack_bf16(lost(r4[2], w[3], 0), lost(r4[3], w[3], 1));
            }
        }

        // values: O^T[16 columns][16 rows] += V^T P^T, two terms of the weights in one instruction
        constexpr int GRP = EXACT ? 4 : 1;     // (the two instructions on one accumulator stand apart)
#pragma unroll
        for (int c0 = 0; c0 < CB; c0 += GRP) {
            bf16x8 a[GRP];
#pragma unroll
            for (int x = 0; x < GRP; ++x) {
                const int cb = c0 + x;
                const char *va = tile + vrd[cb & 3] + (cb >> 2) * 128;
                const s16x4 v4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(va));
                const u32x2 v2 = __builtin_bit_cast(u32x2, v4);
                u32x4 a4;
                a4[0] = v2[0]; a4[1] = v2[1]; a4[2] = v2[0]; a4[3] = v2[1];
                a[x] = __builtin_bit_cast(bf16x8, a4);
            }
#pragma unroll
            for (int x = 0; x < GRP; ++x)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) o[mb][c0 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], pb[mb], o[mb][c0 + x], 0, 0, 0);
            // (half of this one's contraction is zeros; the shorter 16x16x16 must not follow on the same accumulators:
            // a gap of a few instructions between the two shapes lost results of the first)
            if constexpr (EXACT) {
#pragma unroll
                for (int x = 0; x < GRP; ++x) o[0][c0 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], __builtin_bit_cast(bf16x8, w3), o[0][c0 + x], 0, 0, 0);
            }
        }
        // every LDS read of this stage is done before the next iteration's copies may land in it
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        st = st + 1 < NST ? st + 1 : 0;
    }

    // ---- the four waves' partial results meet in LDS ------------------------------------------------------
    float *ml = (float *)(smem + C::OFF_ML);
    uint32_t *odd = (uint32_t *)(smem + C::OFF_ODD);
    constexpr bool CHECK = EXACT && !ALIAS;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
    if (mb > 0) __syncthreads();                   // (the block before has been read)
    {
        float l = l_run[mb];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (j4 == 0) {
            ml[(wave * 16 + n16) * 2] = m_ref[mb];
            ml[(wave * 16 + n16) * 2 + 1] = l;
        }
    }
    {
        char *op = smem + wave * C::REGION + n16 * C::OROW + j4 * 16;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) *(f32x4 *)(op + cb * 64) = o[mb][cb];
    }
    if (CHECK && tid == 0) *odd = 0;
    __syncthreads();
    // wave w finishes rows 4 w .. 4 w + 3 of the block, 512 (or 4 x 128) columns at a time
    // (a lane's columns c .. c + 3 of either half of the row: reads of 16 bytes a lane side by side, whole lines stored)
    constexpr int LPR = DV / 8, RPI = 64 / LPR, HALF = DV / 2;   // lanes per row (8 columns each), rows per step
#pragma unroll
    for (int step = 0; step < 4 / RPI; ++step) {
        const int rr = wave * 4 + step * RPI + lane / LPR, c = (lane % LPR) * 4;
        const int64_t row = r0 + mb * 16 + rr;
        if (row >= R) continue;
        float mw[C::NW], m_all = LOZA_NEG_INF, l_all = 0.f;
#pragma unroll
        for (int w = 0; w < C::NW; ++w) {
            mw[w] = ml[(w * 16 + rr) * 2];
            m_all = fmaxf(m_all, mw[w]);
        }
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
        for (int w = 0; w < C::NW; ++w) {
            const float a = mw[w] == LOZA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(mw[w] - m_all);
            l_all += a * ml[(w * 16 + rr) * 2 + 1];
            const char *op = smem + w * C::REGION + rr * C::OROW + c * 4;
            lo += a * *(const f32x4 *)op;
            hi += a * *(const f32x4 *)(op + HALF * 4);
        }
        const int64_t qi = row_position(row, G);
        const int64_t h = (int64_t)g * G + (row - qi * G);
        const int64_t o_row = ((int64_t)b * Sq + qi) * p.Hq + h;
        if (n_splits > 1) {
            float *po = p.part_o + (o_row * n_splits + split) * DV + c;
            *(f32x4 *)po = lo;
            *(f32x4 *)(po + HALF) = hi;
            if (c == 0) {
                float *pm = p.part_ml + (o_row * n_splits + split) * 4;
                pm[0] = m_all;
                pm[1] = l_all;
            }
            continue;
        }
        const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;   // a row without a live key gives 0
        lo *= inv;
        hi *= inv;
        if (p.out_f32) {
            *(f32x4 *)(p.out_f32 + o_row * DV + c) = lo;
            *(f32x4 *)(p.out_f32 + o_row * DV + c + HALF) = hi;
        } else {
            u32x2 w;
            w[0] = pack_bf16(lo[0], lo[1]);
            w[1] = pack_bf16(lo[2], lo[3]);
            *(u32x2 *)(p.out + o_row * DV + c) = w;
            w[0] = pack_bf16(hi[0], hi[1]);
            w[1] = pack_bf16(hi[2], hi[3]);
            *(u32x2 *)(p.out + o_row * DV + c + HALF) = w;
        }
        if constexpr (CHECK) {
            float z = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) z += lo[e] * 0.f + hi[e] * 0.f;
            if (z != 0.f) atomicOr(odd, 1u << rr);
        }
        if (c == 0) p.lse[((int64_t)b * p.Hq + h) * Sq + qi] = (m_all + __builtin_amdgcn_logf(l_all)) * 0.69314718055994530942f;
    }
    }
    if constexpr (CHECK) {
        // An infinite value at a live key gives an infinity, but the lower terms of its weight may be 0 or negative
        // and made it a NaN (so does the weight 0 of a masked key): such a query is computed again in fp32. (Where
        // the values are part of the keys the score of such a key is not finite either, and a NaN is the result.)
        if (n_splits == 1) {
            lds_barrier();                         // (the stores of the results may still be on their way)
            uint32_t left = *(volatile uint32_t *)odd;
            if (left != 0) {                       // (what has been stored of those rows arrives first)
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                __syncthreads();
            }
            for (; left != 0; left &= left - 1) {
                const int64_t h = (int64_t)b * p.Hq + (int64_t)g * G + r0 + __builtin_ctz(left);
                decode_row_direct<DQK, DV>(p, h, decode_keys(p, h));
                __syncthreads();
            }
        }
    }
}

}  // namespace loza
#endif
