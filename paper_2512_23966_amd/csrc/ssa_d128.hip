// bf16 streaming sparse attention, heads of width 128, many query rows (gfx950): prefill and extend.
//
// Same operation, live keys and two-term rules as ssa_bf16.hip (key tiles of 64; the softmax reference is exact
// over the first 32 keys and then moves when exceeded by 2^8). At this width a key tile
// brings little matrix work per score (a quarter of the absorbed-MLA shape), so the kernel there, whose
// scores change waves between the two products, was bound by LDS traffic and instruction issue: P written
// and read through LDS, every key fragment read for 32 rows (2770 cycles per 32 keys and two workgroups of
// 128 rows, of which 1024 matrix cycles a SIMD). Here
//   * a wave owns 64 query rows (two blocks of 32) through both products: every fragment of a key or value
//     row that comes from LDS feeds two matrix instructions, and the four waves share the staged tile;
//   * P stays in registers: S^T[32 keys][32 rows] = K Q^T leaves lane (h, n) with row n's scores of keys
//     8 x + 4 h + 0 .. 3, the order of the contraction of O^T += V^T P^T is free, and so the eight weights a
//     lane holds for 16 keys are its B operand, and the transposing value reads fetch the keys in that order;
//   * the sum of the rounded weights (the normaliser of O) comes from the matrix core, too: one more column
//     block of ones;
//   * what is left: without the weights 1900 of the 2400 cycles remain, without the fragment reads 2190, without
//     the copies 2190, without mask and check 2020; all of these gone, the 36 matrix instructions take 1310. The
//     wave issues one instruction at a time, and every one costs;
//   * one wave per SIMD, so the two pipes overlap inside the wave: the instruction order of a 32-key step is
//     written out below, one matrix instruction per slot with a few vector instructions in its shadow. While
//     the scores of step u + 1 are taken, the second half of step u's weights is formed; while the values of
//     step u are accumulated, the first half of step u + 1's (against the current reference: that exceeds it
//     by 2^8 is checked before, and almost never so past the first step).
// Keys travel in stages of 64, global -> LDS by global_load_lds_dwordx4 into a ring of four, one barrier per
// stage. A stage holds unpadded rows of 256 bytes whose 16-byte chunks are permuted within groups of eight
// (chunk c of row r in slot c ^ (r & 7)): both kinds of reads are free of bank conflicts.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

namespace {

// One global -> LDS copy instruction (1 KB), unknown to the compiler's wait counters. It names no memory as
// clobbered: what it fills is read only behind a later barrier, and reads of other stages may move across it.
__device__ __forceinline__ void copy_1k(const char *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base), "s"(lds_addr) : "m0");
}

// The matrix instructions of the scores are spelled out to say which half of the register file their operands
// live in (left to itself the compiler accumulates them in AGPRs and copies every one back): scores and the
// queries of the second row block in VGPRs, those of the first in AGPRs, which the output accumulators leave
// room for. The s_nop covers an operand that a vector instruction has just written; whoever reads a result in
// a vector instruction leaves it the time of several matrix instructions, or 24 wait states.
template <int RB>
__device__ __forceinline__ void mfma_first(f32x16 &s, bf16x8 a, bf16x8 b)
{
    if constexpr (RB == 0) asm volatile("s_nop 1\n v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "a"(b));
    else asm volatile("s_nop 1\n v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "v"(b));
}
template <int RB>
__device__ __forceinline__ void mfma_next(f32x16 &s, bf16x8 a, bf16x8 b)
{
    if constexpr (RB == 0) asm volatile("s_nop 1\n v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "a"(b));
    else asm volatile("s_nop 1\n v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "v"(b));
}
}  // namespace

template <bool ALIAS>
struct D128Cfg {
    static constexpr int D = 128, N = 64, SUB = 32, NW = 4, RB = 2;   // keys per stage, per step; row blocks per wave
    static constexpr int M = NW * RB * 32;                            // query rows per workgroup
    static constexpr int ROW = D * 2;                                 // LDS bytes per key row
    static constexpr int KBYTES = N * ROW, STAGE = ALIAS ? KBYTES : 2 * KBYTES;
    static constexpr int NST = 4;
    static constexpr int CP = STAGE / 1024 / NW;                      // copy instructions per wave and stage
    static constexpr int OUTROW = D * 2 + 16;                         // LDS bytes per finished row
    static constexpr int OUTBYTES = M * OUTROW;
    static constexpr int OFF_REDO = NST * STAGE > OUTBYTES ? NST * STAGE : OUTBYTES;
    static constexpr int LDS_BYTES = OFF_REDO + 16;
    static_assert(LDS_BYTES <= 160 * 1024, "does not fit the 160 KB LDS");
};

// One pass over one workgroup tile. PRECISE: two-term weights. Returns true (the same in every wave) when the
// tile has been left unwritten for a PRECISE pass.
template <bool ALIAS, bool PRECISE, bool OUTF32>
static __device__ __forceinline__ bool ssa_d128_tile(const FwdParams &p, char *smem)
{
    using C = D128Cfg<ALIAS>;
    constexpr int M = C::M, N = C::N, NST = C::NST, D = C::D, ROW = C::ROW, RB = C::RB;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, lh = lane >> 5;

    // ---- which tile of which (batch, kv head): every XCD takes one contiguous eighth (see ssa_bf16.hip) ----
    int id = blockIdx.x;
    {
        const int total = gridDim.x, chunk = total / 8;
        if (id < chunk * 8) id = (id % 8) * chunk + id / 8;
    }
    const int rt = p.row_tiles - 1 - id % p.row_tiles;   // heaviest (latest) row tiles first
    id /= p.row_tiles;
    const int g = id % p.Hkv, b = id / p.Hkv, G = p.G;
    const bool cached = p.seqlens != nullptr;            // extend: queries are the last q_len positions of a cache
    const int64_t L = cached ? ((int64_t)p.seqlens[b] < p.S ? (int64_t)p.seqlens[b] : p.S) : p.S;
    const int64_t Sq = cached ? (int64_t)p.q_len : p.S, pos0 = L - Sq, R = Sq * G, r0 = (int64_t)rt * M;
    const int n_sink = p.n_sink, window = p.window, block = p.block;
    auto last_row = [&](int64_t a, int n) { return a + n - 1 < R ? a + n - 1 : R - 1; };
    const int i_min = (int)(pos0 + row_position(r0, G)), i_max = (int)(pos0 + row_position(last_row(r0, M), G));
    if (!PRECISE && i_min < kPrecisePositions) return true;

    // positions of this wave's rows
    const int64_t w0 = r0 + wave * 64 < R ? r0 + wave * 64 : R - 1;
    const int wi_min = (int)(pos0 + row_position(w0, G)), wi_max = (int)(pos0 + row_position(last_row(w0, 64), G));
    const int w_lo_max = window_begin_of(wi_max < 0 ? 0 : wi_max, window, block);

    // ---- live key tiles of 64: sink tiles [0, nA), then window tiles [wt0, wt0 + nB) in rotated order -------
    const int sink_end = i_max < 0 ? 0 : (n_sink < i_max + 1 ? n_sink : i_max + 1);
    const int win_begin = window_begin_of(i_min < 0 ? 0 : i_min, window, block);
    int nA = (sink_end + N - 1) / N;
    const int wt0 = win_begin / N, wt1 = i_max / N;
    int nB;
    if (wt0 <= nA) { nA = wt1 + 1; nB = 0; } else { nB = wt1 - wt0 + 1; }
    if (i_max < 0) { nA = 0; nB = 0; }
    const int nt = nA + nB;
    int w_rot = 0;
    if (nB > 1) { w_rot = wt0 % nB; w_rot = w_rot == 0 ? 0 : nB - w_rot; }
    auto key_tile = [&](int t) {
        if (t < nA) return t;
        int x = t - nA + w_rot;
        x = x >= nB ? x - nB : x;
        return wt0 + x;
    };

    // ---- copies: a stage is two halves of 32 rows (a page holds at least 32); instruction x of a half's eight
    // moves rows 4 x .. 4 x + 3 and belongs to wave x % 4, so a wave's rows are 4 wave + lane / 16 (+ 16) -------
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const uint32_t stride = (uint32_t)p.Hkv * ROW;       // keys and values alike
    const int c_row = wave * 4 + (lane >> 4);
    const uint32_t c_chunk = (uint32_t)((lane & 8) | ((lane ^ c_row) & 7)) * 16u;
    const bool paged = p.block_table != nullptr;
    const int64_t seq_row0 = paged ? 0 : (int64_t)b * p.S;
    const char *kbase = (const char *)p.k + (seq_row0 * p.Hkv + g) * (int64_t)ROW;
    const char *vbase = (const char *)p.v + (seq_row0 * p.Hkv + g) * (int64_t)ROW;
    const i32x4 table_rsrc = paged ? table_row_resource(p.block_table + (int64_t)b * p.max_pages, p.max_pages) : i32x4{0, 0, 0, 0};
    struct StageCopy {
        int64_t row[2];    // cache row a half starts at, relative to kbase / vbase (in rows)
        int lim[2];        // its last valid row
        uint32_t dst;
    };
    auto plan_stage = [&](int t, int slot) {
        StageCopy sc;
        const int j0 = key_tile(t) * N;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // A half without a live key of this row tile (between the sink and the first window key, or past the
            // last query) is never read: its page may be evicted or stale, and weight 0 times a NaN is a NaN. The
            // stage's other half, which has one, is copied in its place, and masked there.
            const int jh = j0 + 32 * h;
            const bool live = jh < sink_end || (jh + 31 >= win_begin && jh <= i_max);
            const int j = live ? jh : j0 + 32 * (1 - h);
            const int left = (int)(L - 1) - j;
            sc.lim[h] = left < 31 ? left : 31;
            sc.row[h] = j;
            if (paged) {
                int32_t pid = llvm_amdgcn_s_buffer_load_i32(table_rsrc, (int32_t)((uint32_t)(j >> p.page_shift) * 4u), 0);
                pid = pid < 0 ? 0 : (pid < p.num_pages ? pid : p.num_pages - 1);   // a bad entry stays in bounds
                sc.row[h] = ((int64_t)pid << p.page_shift) + (j & ((1 << p.page_shift) - 1));
            }
        }
        sc.dst = smem_lds + slot * C::STAGE + wave * 1024;
        return sc;
    };
    // copy instruction c of this wave (a constant after unrolling): half c / 4 (aliased: c / 2), ...
    auto copy_nth = [&](const StageCopy &sc, int c) {
        constexpr int PER = C::CP / 2;
        const int h = c / PER, y = c % PER, x = ALIAS ? y : y >> 1, is_v = ALIAS ? 0 : y & 1;
        const int row = c_row + 16 * x;
        const uint32_t off = (uint32_t)(row < sc.lim[h] ? row : sc.lim[h]) * stride + c_chunk;
        copy_1k((is_v ? vbase : kbase) + sc.row[h] * (int64_t)stride, off, sc.dst + (is_v ? C::KBYTES : 0) + h * 8192 + x * 4096);
    };
    auto copy_stage = [&](const StageCopy &sc) {
#pragma unroll
        for (int c = 0; c < C::CP; ++c) copy_nth(sc, c);
    };
    if (nt > 0) copy_stage(plan_stage(0, 0));

    // ---- the queries: B operands, row ln of each block ------------------------------------------------------
    bf16x8 qf[RB][8];
    int i_row[RB], w_lo_row[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int64_t row = r0 + wave * 64 + rb * 32 + ln, rc = row < R ? row : R - 1, qi = row_position(rc, G);
        i_row[rb] = (int)(pos0 + qi);
        w_lo_row[rb] = window_begin_of(i_row[rb] < 0 ? 0 : i_row[rb], window, block);
        const uint16_t *qp = p.q + (((int64_t)b * Sq + qi) * p.Hq + (int64_t)g * G + (rc - qi * G)) * D + lh * 8;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[rb][kk] = *(const bf16x8 *)(qp + kk * 16);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // (with a wait the compiler sees; the first stage has landed, too)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        asm volatile("" : "+a"(qf[0][kk]));
        asm volatile("" : "+v"(qf[1][kk]));
    }
    // (every stage is copied, also those past the last: the wait counts are the same throughout)
    if (nt > 0) {
#pragma unroll
        for (int a = 1; a < NST - 1; ++a) copy_stage(plan_stage(a < nt ? a : nt - 1, a));
    }
    int *s_redo = (int *)(smem + C::OFF_REDO);
    if (!PRECISE && tid == 0) *s_redo = 0;
    lds_barrier();

    // ---- state ---------------------------------------------------------------------------------------------
    f32x16 o[RB][4], osum[RB];                  // O^T, and the sum of the rounded weights in every element
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            osum[rb][e] = 0.f;
#pragma unroll
            for (int db = 0; db < 4; ++db) o[rb][db][e] = 0.f;
        }
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    float m_ref[RB], m_use[RB], l_run[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_ref[rb] = LOZA_NEG_INF;
        m_use[rb] = 0.f;
        l_run[rb][0] = l_run[rb][1] = 0.f;
    }
    // LDS offsets of this lane's reads within a step's 32 rows (keys: row ln; values: rows 4 lh + ..., transposing)
    uint32_t krd[4], vrd[2];
#pragma unroll
    for (int x = 0; x < 4; ++x) krd[x] = (uint32_t)(ln * ROW + (((x * 2 + lh) ^ (ln & 7)) * 16));
    {
        const int s16 = lane & 15, g16 = (lane >> 4) & 1, vr = lh * 4 + (s16 >> 2);
#pragma unroll
        for (int x = 0; x < 2; ++x)
            vrd[x] = (uint32_t)((ALIAS ? 0 : C::KBYTES) + vr * ROW + (((x * 4 + g16 * 2 + ((s16 & 3) >> 1)) ^ (vr & 7)) * 16) + (s16 & 1) * 8);
    }
    auto read_k = [&](const char *kt, int kk) { return *(const bf16x8 *)(kt + krd[kk & 3] + (kk >> 2) * 128); };
    auto read_v = [&](const char *vt, int f) {   // fragment f = ks * 4 + db
        const char *a = vt + vrd[f & 1] + ((f >> 1) & 1) * 128 + (f >> 2) * 16 * ROW;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a + 8 * ROW));
        s16x8 a8;
        a8[0] = lo[0]; a8[1] = lo[1]; a8[2] = lo[2]; a8[3] = lo[3];
        a8[4] = hi[0]; a8[5] = hi[1]; a8[6] = hi[2]; a8[7] = hi[3];
        return __builtin_bit_cast(bf16x8, a8);
    };
    // address of step u (32 keys): half u & 1 of stage (u >> 1) % NST
    auto step_tile = [&](int u) { return (const char *)smem + ((u >> 1) & (NST - 1)) * C::STAGE + (u & 1) * 32 * ROW; };
    auto step_key = [&](int u) { return (u >> 1) < nt ? key_tile(u >> 1) * N + (u & 1) * 32 : kNoTile; };

    f32x16 s[2][RB];                            // scores of the steps of either parity, exponentials in place
    u32x4 pk[2][2][RB];                         // [parity][key half]: rounded weights, B operands
    u32x4 pl[PRECISE ? 2 : 1][2][RB];           // what the rounding lost
    auto mask = [&](f32x16 (&x)[RB], int j0) {
        const bool interior = (j0 + 31 <= wi_min) && ((j0 + 31 < n_sink) || (j0 >= w_lo_max));
        if (!interior) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int j = j0 + 4 * lh + 8 * (e >> 2) + (e & 3);
                    const bool ok = (j <= i_row[rb]) & ((j < n_sink) | (j >= w_lo_row[rb]));
                    x[rb][e] = ok ? x[rb][e] : LOZA_NEG_INF;
                }
        }
    };
    float alpha[RB];
    // the reference moves: every row takes its running maximum (mx: of this lane's 16 scores, unscaled)
    auto move_reference = [&](const float (&mx)[RB]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float m_new = fmaxf(m_ref[rb], max_with_other_half(mx[rb]) * p.scale_log2);   // scale > 0
            alpha[rb] = m_new == LOZA_NEG_INF ? 1.0f : __builtin_amdgcn_exp2f(m_ref[rb] - m_new);
            m_ref[rb] = m_new;
            m_use[rb] = m_new == LOZA_NEG_INF ? 0.f : m_new;   // a row with no live key so far
            l_run[rb][0] *= alpha[rb];
            l_run[rb][1] *= alpha[rb];
        }
    };
    auto rescale = [&]() {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            auto mul = [&](f32x16 &x) {   // (pinned in AGPRs on both sides: moved through VGPRs only here)
                f32x16 t = x;
                asm volatile("" : "+a"(t));
#pragma unroll
                for (int e = 0; e < 16; ++e) t[e] *= alpha[rb];
                asm volatile("" : "+a"(t));
                x = t;
            };
#pragma unroll
            for (int db = 0; db < 4; ++db) mul(o[rb][db]);
            mul(osum[rb]);
        }
    };
    // element j (0 .. 15) of a key half: pairs of one row block, the two row blocks in turn
    auto el_rb = [](int j) { return (j >> 1) & 1; };
    auto el_e = [](int half, int j) { return half * 8 + ((j >> 2) << 1) + (j & 1); };
    // stage (0 scale, 1 exponential, 2 sum and, of a pair's second, pack) of element j
    auto weight = [&](auto par_c, int half, int j, int stage) {
        constexpr int PAR = decltype(par_c)::value;
        if (j < 0 || j >= 16) return;
        const int rb = el_rb(j), e = el_e(half, j);
        f32x16 &x = s[PAR][rb];
        // (the empty asm statements anchor each result in its slot: the optimiser otherwise sinks all of this
        // arithmetic below the last matrix instruction)
        if (stage == 0) {
            x[e] = __builtin_fmaf(x[e], p.scale_log2, -m_use[rb]);
            asm volatile("" : "+v"(x));
        } else if (stage == 1) {
            x[e] = __builtin_amdgcn_exp2f(x[e]);
            asm volatile("" : "+v"(x));
        } else {
            l_run[rb][e & 1] += x[e];
            asm volatile("" : "+v"(l_run[rb][e & 1]));
            if (e & 1) {
                const int w = (e & 7) >> 1;
                pk[PAR][half][rb][w] = pack_bf16(x[e - 1], x[e]);
                asm volatile("" : "+v"(pk[PAR][half][rb]));
                if constexpr (PRECISE) {
                    const uint32_t q = pk[PAR][half][rb][w];
                    pl[PAR][half][rb][w] = pack_bf16(x[e - 1] - __builtin_bit_cast(float, q << 16), x[e] - __builtin_bit_cast(float, q & 0xffff0000u));
                }
            }
        }
    };

    auto score = [&](f32x16 &x, int rb, int kk, bf16x8 a) {
        if (rb == 0) {
            if (kk == 0) mfma_first<0>(x, a, qf[0][kk]);
            else mfma_next<0>(x, a, qf[0][kk]);
        } else {
            if (kk == 0) mfma_first<1>(x, a, qf[1][kk]);
            else mfma_next<1>(x, a, qf[1][kk]);
        }
    };
    if (nt > 0) {
        // ---- first step: scores, reference, first half of its weights -----------------------------------------
        bf16x8 kf[4];
        {
            const char *kt = step_tile(0);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const bf16x8 a = read_k(kt, kk);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    score(s[0][rb], rb, kk, a);
                }
            }
            asm volatile("s_nop 7\n s_nop 7\n s_nop 7" : "+v"(s[0][0]), "+v"(s[0][1]));
            mask(s[0], step_key(0));
            float mx[RB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                mx[rb] = s[0][rb][0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx[rb] = fmaxf(mx[rb], s[0][rb][e]);
            }
            move_reference(mx);
#pragma unroll
            for (int j = 0; j < 16; ++j)
#pragma unroll
                for (int st = 0; st < 3; ++st) weight(std::integral_constant<int, 0>{}, 0, j, st);
            const char *k1 = step_tile(1);
#pragma unroll
            for (int x = 0; x < 3; ++x) kf[x] = read_k(k1, x);
        }

        // ---- one step of 32 keys: values of step u, scores of step u + 1 --------------------------------------
        auto step = [&](auto par_c, const int u, const StageCopy &sc) {
            constexpr int PAR = decltype(par_c)::value, NPAR = PAR ^ 1;
            using P = std::integral_constant<int, PAR>;
            using Q = std::integral_constant<int, NPAR>;
            const char *kt = step_tile(u + 1), *k2 = step_tile(u + 2), *vt = step_tile(u);
            bf16x8 vf[4];
            float mx[RB];
            bool moved = false;
            // slots 0 .. 15: scores of u + 1; the second half of u's weights (element j: scaled in slot j,
            // exponentiated in j + 1, summed and packed in j + 2)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int kk = i >> 1, rb = i & 1;
                score(s[NPAR][rb], rb, kk, kf[kk & 3]);
                if (rb == 0) kf[(kk + 3) & 3] = kk + 3 < 8 ? read_k(kt, kk + 3) : read_k(k2, kk + 3 - 8);
                weight(P{}, 1, i - 2, 2);
                weight(P{}, 1, i - 1, 1);
                weight(P{}, 1, i, 0);
                if (i == 9) vf[0] = read_v(vt, 0);
                if (i == 11) vf[1] = read_v(vt, 1);
                if (i == 13) vf[2] = read_v(vt, 2);
                if (PAR == 0 && (i & 1) && (i >> 1) < C::CP) copy_nth(sc, i >> 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            // slots 16 .. 35: values of u (per key half: four column blocks and the ones, both row blocks)
            auto value = [&](int x) {
                const int ks = x / 10, y = x % 10, rb = y & 1, db = y >> 1, f = ks * 4 + db;
                const bf16x8 ph = __builtin_bit_cast(bf16x8, pk[PAR][ks][rb]);
                if (y < 8) {
                    o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f & 3], ph, o[rb][db], 0, 0, 0);
                    if constexpr (PRECISE) o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f & 3], __builtin_bit_cast(bf16x8, pl[PAR][ks][rb]), o[rb][db], 0, 0, 0);
                    if (rb == 0 && f + 3 < 8) vf[(f + 3) & 3] = read_v(vt, f + 3);
                } else {
                    osum[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, ph, osum[rb], 0, 0, 0);
                    if constexpr (PRECISE) osum[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, __builtin_bit_cast(bf16x8, pl[PAR][ks][rb]), osum[rb], 0, 0, 0);
                }
            };
            weight(P{}, 1, 14, 2);
            weight(P{}, 1, 15, 1);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                value(x);
                if (x == 0) weight(P{}, 1, 15, 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the scores of u + 1 have left the matrix pipeline (four matrix instructions ago)
            asm volatile("s_nop 3" : "+v"(s[NPAR][0]), "+v"(s[NPAR][1]));
            mask(s[NPAR], step_key(u + 1));
#pragma unroll
            for (int x = 4; x < 8; ++x) {
                value(x);
                const int rb = (x - 4) >> 1, h = (x & 1) * 8;
                float m8 = fmaxf(fmaxf(s[NPAR][rb][h], s[NPAR][rb][h + 1]), s[NPAR][rb][h + 2]);
                m8 = fmaxf(fmaxf(m8, s[NPAR][rb][h + 3]), s[NPAR][rb][h + 4]);
                m8 = fmaxf(fmaxf(m8, s[NPAR][rb][h + 5]), s[NPAR][rb][h + 6]);
                m8 = fmaxf(m8, s[NPAR][rb][h + 7]);
                mx[rb] = h == 0 ? m8 : fmaxf(mx[rb], m8);
                asm volatile("" : "+v"(mx[rb]));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (__any((mx[0] * p.scale_log2 > m_ref[0] + p.lazy_log2) | (mx[1] * p.scale_log2 > m_ref[1] + p.lazy_log2))) {
                move_reference(mx);
                moved = true;
            }
            // slots 24 .. 35, and the first half of u + 1's weights
#pragma unroll
            for (int x = 8; x < 20; ++x) {
                value(x);
                const int a = (x - 8) * 4 / 3, z = (x - 7) * 4 / 3;   // elements scaled in this slot
                const int a1 = (x - 9) * 4 / 3, a2 = (x - 10) * 4 / 3;
                if (x >= 10) {
#pragma unroll
                    for (int j = a2; j < a1; ++j) weight(Q{}, 0, j, 2);
                }
                if (x >= 9) {
#pragma unroll
                    for (int j = a1; j < a; ++j) weight(Q{}, 0, j, 1);
                }
#pragma unroll
                for (int j = a; j < z; ++j) weight(Q{}, 0, j, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 14; j < 16; ++j) weight(Q{}, 0, j, 1);
#pragma unroll
            for (int j = 13; j < 16; ++j) weight(Q{}, 0, j, 2);
            if (moved) rescale();
        };
        for (int t = 0; t < nt; ++t) {
            // stage t + 1 has landed when at most the copies of the stages after it are outstanding; the stage
            // of t - 1 is no longer read (past the last stage the current one, hot in L2, is copied again)
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 3) * C::CP) : "memory");
            lds_barrier();
            // (the accumulators cross the loop in AGPRs: without this the rescale path, which needs them in VGPRs,
            // decides, and they are moved back and forth every time)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int db = 0; db < 4; ++db) asm volatile("" : "+a"(o[rb][db]));
                asm volatile("" : "+a"(osum[rb]));
            }
            const StageCopy sc = plan_stage(t + NST - 1 < nt ? t + NST - 1 : t, (t + NST - 1) & (NST - 1));
            step(std::integral_constant<int, 0>{}, 2 * t, sc);
            step(std::integral_constant<int, 1>{}, 2 * t + 1, sc);
        }
    }

    // ---- epilogue --------------------------------------------------------------------------------------------
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may be on its way into LDS any more
    lds_barrier();                                     // the stages are no longer read
    bool big = false;
    float inv[RB], lse[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float l1 = l_run[rb][0] + l_run[rb][1], l = l1 + xor32(l1);
        lse[rb] = (m_ref[rb] + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
        inv[rb] = osum[rb][0] > 0.f ? 1.0f / osum[rb][0] : 0.f;   // a row without a live key gives 0
        const int row = wave * 64 + rb * 32 + ln;
        float mx = 0.f;
        char *op = smem + row * C::OUTROW + lh * 8;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = o[rb][db][4 * qd + e] * inv[rb];
                    if (!PRECISE) mx = fmaxf(mx, __builtin_fabsf(x[e]));
                }
                if constexpr (!OUTF32) {
                    u32x2 w;
                    w[0] = pack_bf16(x[0], x[1]);
                    w[1] = pack_bf16(x[2], x[3]);
                    *(u32x2 *)(op + db * 64 + qd * 16) = w;
                }
            }
        big = big || (mx >= kRedoMagnitude && r0 + row < R);
    }
    if (!PRECISE) {
        if (__any(big) && lane == 0) *s_redo = 1;
        lds_barrier();
        if (*(volatile int *)s_redo) return true;
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int64_t row = r0 + wave * 64 + rb * 32 + ln;
        if (row < R) {
            const int64_t i = row_position(row, G);
            const int64_t h = (int64_t)g * G + (row - i * G);
            if (lh == 0) p.lse[((int64_t)b * p.Hq + h) * Sq + i] = lse[rb];
            if constexpr (OUTF32) {
                // unrounded output (the calibration blend rounds once, after mixing two of these)
                float *op = p.out_f32 + (((int64_t)b * Sq + i) * p.Hq + h) * D + 4 * lh;
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) {
                        float4 w;
                        w.x = o[rb][db][4 * qd + 0] * inv[rb];
                        w.y = o[rb][db][4 * qd + 1] * inv[rb];
                        w.z = o[rb][db][4 * qd + 2] * inv[rb];
                        w.w = o[rb][db][4 * qd + 3] * inv[rb];
                        *(float4 *)(op + db * 32 + qd * 8) = w;
                    }
            }
        }
    }
    if constexpr (!OUTF32) {
        // (a wave stores its own rows: four of them an instruction)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int first = wave * 64 + (lane >> 4);
        int64_t i = row_position(r0 + first, G);
        int hh = (int)(r0 + first - i * G);
#pragma unroll 4
        for (int st = 0; st < 16; ++st) {
            const int row = first + st * 4;
            if (r0 + row < R) {
                const u32x4 w = *(const u32x4 *)(smem + row * C::OUTROW + (lane & 15) * 16);
                const int64_t o_row = ((int64_t)b * Sq + i) * p.Hq + (int64_t)g * G + hh;
                __builtin_nontemporal_store(w, (u32x4 *)(p.out + o_row * D + (lane & 15) * 8));
            }
            hh += 4;
            if (hh >= G) {
                const int d = hh / G;
                i += d;
                hh -= d * G;
            }
        }
    }
    return false;
}

template <bool ALIAS, bool OUTF32>
__global__ __launch_bounds__(256) void ssa_d128_kernel(const FwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    if (ssa_d128_tile<ALIAS, false, OUTF32>(p, smem)) ssa_d128_tile<ALIAS, true, OUTF32>(p, smem);
}

template <bool ALIAS, bool OUTF32>
static hipError_t launch_d128_t(FwdParams p, hipStream_t stream)
{
    using C = D128Cfg<ALIAS>;
    constexpr auto kern = ssa_d128_kernel<ALIAS, OUTF32>;
    hipError_t e = allow_lds<kern>(C::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int64_t rows = (p.seqlens ? (int64_t)p.q_len : p.S) * p.G;
    p.row_tiles = (int)((rows + C::M - 1) / C::M);
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)p.row_tiles * p.Hkv * p.B)), dim3(256), C::LDS_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_d128_bf16(const FwdParams &p, bool alias, hipStream_t stream)
{
    if (p.out_f32 != nullptr) return alias ? launch_d128_t<true, true>(p, stream) : launch_d128_t<false, true>(p, stream);
    return alias ? launch_d128_t<true, false>(p, stream) : launch_d128_t<false, false>(p, stream);
}

}  // namespace loza
