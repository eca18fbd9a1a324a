// bf16 streaming sparse attention, heads of width 128, many query rows (gfx950): prefill and extend.
//
// Same operation, live keys and two-term rules as ssa_bf16.hip (key tiles of 64; the softmax reference is exact
// over the first 32 live keys and then moves when exceeded by 2^8). At this width a key tile
// brings little matrix work per score (a quarter of the absorbed-MLA shape), so the kernel there, whose
// scores change waves between the two products, was bound by LDS traffic and instruction issue: P written
// and read through LDS (2770 cycles per 32 keys and two workgroups of
// 128 rows, of which 1024 matrix cycles a SIMD). Here
//   * a wave owns 32 query rows through both products, and the eight waves of a workgroup share the staged tile;
//   * P stays in registers: S^T[32 keys][32 rows] = K Q^T leaves lane (h, n) with row n's scores of keys
//     8 x + 4 h + 0 .. 3, the order of the contraction of O^T += V^T P^T is free, and so the eight weights a
//     lane holds for 16 keys are its B operand, and the transposing value reads fetch the keys in that order;
//   * the sum of the rounded weights (the normaliser of O) comes from the matrix core, too: one more column
//     block of ones;
//   * two waves per SIMD: one's matrix instructions run while the other forms exponentials or waits for LDS: 1152 cycles of
//     matrix work a step of 32 keys and SIMD in about 1900, and nearly as many of vector work; the LDS is busy for 20 % of
//     them. (Four waves of 64 rows, one a SIMD, issue one instruction at a time: interleaved by hand, one matrix
//     instruction per slot, a step took 2400 cycles.)
// Keys travel in stages of 64, global -> LDS by global_load_lds_dwordx4 into a ring of four, one barrier per
// stage. A stage holds unpadded rows of 256 bytes whose 16-byte chunks are permuted (row_swizzle) so that both kinds of
// reads are free of bank conflicts. (Permuted within groups of eight, by c ^ (r & 7), the four rows of a transposing read lay
// in the same 16 banks and rows r and r + 8 of the other kind in the same four: two thirds of the LDS's cycles were
// conflicts, 59 % of all cycles LDS. 32 heads of their own keys, 32,768 tokens: 2262 us, now 2212.)
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

}  // namespace

template <bool ALIAS>
struct D128Cfg {
    static constexpr int D = 128, N = 64, NW = 8;   // keys per stage; waves
    static constexpr int M = NW * 32;                                 // query rows per workgroup
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
    constexpr int M = C::M, N = C::N, NST = C::NST, D = C::D, ROW = C::ROW;
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
    const int64_t w0 = r0 + wave * 32 < R ? r0 + wave * 32 : R - 1;
    const int wi_min = (int)(pos0 + row_position(w0, G)), wi_max = (int)(pos0 + row_position(last_row(w0, 32), G));
    const int w_lo_min = window_begin_of(wi_min < 0 ? 0 : wi_min, window, block);
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
    // moves rows 4 x .. 4 x + 3 and belongs to wave x, so a wave's rows are 4 wave + lane / 16 -------------------
    const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);
    const uint32_t stride = (uint32_t)p.Hkv * ROW;       // keys and values alike
    const int c_row = wave * 4 + (lane >> 4);
    const uint32_t c_chunk = ((uint32_t)(lane & 15) ^ row_swizzle(c_row)) * 16u;
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
    // copy instruction c of this wave (a constant after unrolling): half c / 2 (aliased: c), keys, then values
    auto copy_nth = [&](const StageCopy &sc, int c) {
        constexpr int PER = C::CP / 2;
        const int h = c / PER, is_v = c % PER;
        const uint32_t off = (uint32_t)(c_row < sc.lim[h] ? c_row : sc.lim[h]) * stride + c_chunk;
        copy_1k((is_v ? vbase : kbase) + sc.row[h] * (int64_t)stride, off, sc.dst + (is_v ? C::KBYTES : 0) + h * 8192);
    };
    auto copy_stage = [&](const StageCopy &sc) {
#pragma unroll
        for (int c = 0; c < C::CP; ++c) copy_nth(sc, c);
    };
    if (nt > 0) copy_stage(plan_stage(0, 0));

    // ---- the queries: B operands, row ln of each block ------------------------------------------------------
    bf16x8 qf[8];
    int i_row, w_lo_row;
    {
        const int64_t row = r0 + wave * 32 + ln, rc = row < R ? row : R - 1, qi = row_position(rc, G);
        i_row = (int)(pos0 + qi);
        w_lo_row = window_begin_of(i_row < 0 ? 0 : i_row, window, block);
        const uint16_t *qp = p.q + (((int64_t)b * Sq + qi) * p.Hq + (int64_t)g * G + (rc - qi * G)) * D + lh * 8;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[kk] = *(const bf16x8 *)(qp + kk * 16);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // (with a wait the compiler sees; the first stage has landed, too)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) asm volatile("" : "+v"(qf[kk]));
    // (every stage is copied, also those past the last: the wait counts are the same throughout)
    if (nt > 0) {
#pragma unroll
        for (int a = 1; a < NST - 1; ++a) copy_stage(plan_stage(a < nt ? a : nt - 1, a));
    }
    int *s_redo = (int *)(smem + C::OFF_REDO);
    if (!PRECISE && tid == 0) *s_redo = 0;
    lds_barrier();

    // ---- state ---------------------------------------------------------------------------------------------
    f32x16 o[4], osum;                          // O^T, and the sum of the rounded weights in every element
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        osum[e] = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db) o[db][e] = 0.f;
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    float m_ref = LOZA_NEG_INF, l_run[2] = {0.f, 0.f};
    // LDS offsets of this lane's reads within 32 rows (keys: row ln; values: rows 4 lh + ..., transposing), of fragment
    // 0; the permutation makes the others' a matter of single bits
    const int s16 = lane & 15, v_row = lh * 4 + (s16 >> 2);
    const uint32_t k_rd = (uint32_t)(ln * ROW) + ((uint32_t)lh ^ row_swizzle(ln)) * 16u;
    const uint32_t v_rd = (uint32_t)((ALIAS ? 0 : C::KBYTES) + v_row * ROW + (s16 & 1) * 8) + ((uint32_t)(((lane >> 4) & 1) * 2 + ((s16 & 3) >> 1)) ^ row_swizzle(v_row)) * 16u;
    auto read_k = [&](uint32_t a, int kk) {
        return *(__attribute__((address_space(3))) const bf16x8 *)(uintptr_t)(a ^ (kk << 5));
    };
    auto read_v = [&](uint32_t a, int f) {       // fragment f = ks * 4 + db
        const uint32_t x = (a ^ ((f & 3) << 6)) + (f >> 2) * 16 * ROW, y = (a ^ ((f & 3) << 6 | 32)) + (f >> 2) * 16 * ROW + 8 * ROW;   // (row r + 8: swizzled by 2 more)
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)x);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)y);
        s16x8 a8;
        a8[0] = lo[0]; a8[1] = lo[1]; a8[2] = lo[2]; a8[3] = lo[3];
        a8[4] = hi[0]; a8[5] = hi[1]; a8[6] = hi[2]; a8[7] = hi[3];
        return __builtin_bit_cast(bf16x8, a8);
    };
    // One step: the 32 keys j0 .., in LDS at `tile`.
    auto step = [&](const int j0, const uint32_t tile) {
        if (j0 > wi_max || (j0 >= n_sink && j0 + 31 < w_lo_min)) return;   // no row of this wave sees any of them
        constexpr int PF = 4;
        f32x16 s;
        __builtin_amdgcn_s_setprio(1);          // (matrix phases first: the other wave of the SIMD fills in)
        {
            uint32_t a = tile + k_rd;
            asm volatile("" : "+v"(a));
            bf16x8 f[PF];
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int m = 0; m < PF; ++m) f[m] = read_k(a, m);
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[m % PF], qf[m], s, 0, 0, 0);
                if (m + PF < 8) f[m % PF] = read_k(a, m + PF);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        const bool interior = (j0 + 31 <= wi_min) && ((j0 + 31 < n_sink) || (j0 >= w_lo_max));
        if (!interior) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int j = j0 + 4 * lh + 8 * (e >> 2) + (e & 3);
                const bool ok = (j <= i_row) & ((j < n_sink) | (j >= w_lo_row));
                s[e] = ok ? s[e] : LOZA_NEG_INF;
            }
        }
        float mx = fmaxf(s[0], s[1]);
#pragma unroll
        for (int e = 2; e < 16; e += 2) mx = fmaxf(fmaxf(mx, s[e]), s[e + 1]);
        if (__any(mx * p.scale_log2 > m_ref + p.lazy_log2)) {
            // the reference moves: every row takes its running maximum
            const float m_new = fmaxf(m_ref, max_with_other_half(mx) * p.scale_log2);   // scale > 0
            const float alpha = m_new == LOZA_NEG_INF ? 1.0f : __builtin_amdgcn_exp2f(m_ref - m_new);
            m_ref = m_new;
            l_run[0] *= alpha;
            l_run[1] *= alpha;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                osum[e] *= alpha;
#pragma unroll
                for (int db = 0; db < 4; ++db) o[db][e] *= alpha;
            }
        }
        const float m_use = m_ref == LOZA_NEG_INF ? 0.f : m_ref;   // a row with no live key so far
        u32x4 pk[2], pl[2];
        uint32_t va = tile + v_rd;
        asm volatile("" : "+v"(va));
        bf16x8 vf[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) vf[f] = read_v(va, f);   // (lands under the exponentials)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], p.scale_log2, -m_use));
            const float b2 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], p.scale_log2, -m_use));
            l_run[0] += a;
            l_run[1] += b2;
            const uint32_t w = pack_bf16(a, b2);
            pk[e >> 3][(e & 7) >> 1] = w;
            if constexpr (PRECISE) pl[e >> 3][(e & 7) >> 1] = pack_bf16(a - __builtin_bit_cast(float, w << 16), b2 - __builtin_bit_cast(float, w & 0xffff0000u));
        }
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const int ks = f >> 2, db = f & 3;
            const bf16x8 ph = __builtin_bit_cast(bf16x8, pk[ks]);
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f % PF], ph, o[db], 0, 0, 0);
            if constexpr (PRECISE) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f % PF], __builtin_bit_cast(bf16x8, pl[ks]), o[db], 0, 0, 0);
            if (f + PF < 8) vf[f % PF] = read_v(va, f + PF);
            if (db == 3) {
                osum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, ph, osum, 0, 0, 0);
                if constexpr (PRECISE) osum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, __builtin_bit_cast(bf16x8, pl[ks]), osum, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    for (int t = 0; t < nt; ++t) {
        // stage t has landed when at most the copies of the stages after it are outstanding; the stage of t - 1 is no
        // longer read (past the last stage the current one, hot in L2, is copied again)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 2) * C::CP) : "memory");
        lds_barrier();
        copy_stage(plan_stage(t + NST - 1 < nt ? t + NST - 1 : t, (t + NST - 1) & (NST - 1)));
        const uint32_t stage = smem_lds + (t & (NST - 1)) * C::STAGE;
        step(key_tile(t) * N, stage);
        step(key_tile(t) * N + 32, stage + 32 * ROW);
    }

    // ---- epilogue --------------------------------------------------------------------------------------------
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may be on its way into LDS any more
    lds_barrier();                                     // the stages are no longer read
    bool big = false;
    float inv, lse;
    {
        const float l1 = l_run[0] + l_run[1], l = l1 + xor32(l1);
        lse = (m_ref + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
        inv = osum[0] > 0.f ? 1.0f / osum[0] : 0.f;   // a row without a live key gives 0
        const int row = wave * 32 + ln;
        float mx = 0.f;
        char *op = smem + row * C::OUTROW + lh * 8;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = o[db][4 * qd + e] * inv;
                    if (!PRECISE) mx = fmaxf(mx, __builtin_fabsf(x[e]));
                }
                if constexpr (!OUTF32) {
                    u32x2 w;
                    w[0] = pack_bf16(x[0], x[1]);
                    w[1] = pack_bf16(x[2], x[3]);
                    *(u32x2 *)(op + db * 64 + qd * 16) = w;
                }
            }
        big = mx >= kRedoMagnitude && r0 + row < R;
    }
    if (!PRECISE) {
        if (__any(big) && lane == 0) *s_redo = 1;
        lds_barrier();
        if (*(volatile int *)s_redo) return true;
    }
    {
        const int64_t row = r0 + wave * 32 + ln;
        if (row < R) {
            const int64_t i = row_position(row, G);
            const int64_t h = (int64_t)g * G + (row - i * G);
            if (lh == 0) p.lse[((int64_t)b * p.Hq + h) * Sq + i] = lse;
            if constexpr (OUTF32) {
                // unrounded output (the calibration blend rounds once, after mixing two of these)
                float *op = p.out_f32 + (((int64_t)b * Sq + i) * p.Hq + h) * D + 4 * lh;
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) {
                        float4 w;
                        w.x = o[db][4 * qd + 0] * inv;
                        w.y = o[db][4 * qd + 1] * inv;
                        w.z = o[db][4 * qd + 2] * inv;
                        w.w = o[db][4 * qd + 3] * inv;
                        *(float4 *)(op + db * 32 + qd * 8) = w;
                    }
            }
        }
    }
    if constexpr (!OUTF32) {
        // (a wave stores its own rows: four of them an instruction)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int first = wave * 32 + (lane >> 4);
        int64_t i = row_position(r0 + first, G);
        int hh = (int)(r0 + first - i * G);
#pragma unroll 4
        for (int st = 0; st < 8; ++st) {
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
__global__ __launch_bounds__(512, 2) void ssa_d128_kernel(const FwdParams p)
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
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)p.row_tiles * p.Hkv * p.B)), dim3(64 * C::NW), C::LDS_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_d128_bf16(const FwdParams &p, bool alias, hipStream_t stream)
{
    if (p.out_f32 != nullptr) return alias ? launch_d128_t<true, true>(p, stream) : launch_d128_t<false, true>(p, stream);
    return alias ? launch_d128_t<true, false>(p, stream) : launch_d128_t<false, false>(p, stream);
}

}  // namespace loza
