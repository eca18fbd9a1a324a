// bf16 streaming sparse attention for few query rows (gfx950): decode, short extends, short prompts. The pass over
// sixteen rows and the reasons for it are in ssa_rows.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssa_device.h"
#include "ssa_direct.h"
#include "ssa_kernels.h"
#include "ssa_rows.h"

namespace loza {

template <int DQK, int DV, bool ALIAS, bool NT, bool EXACT, int MB>
__global__ __launch_bounds__(256) void ssa_rows_kernel(const FwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // ---- which rows of which (batch, kv head), which split -----------------------------------------
    // A unit is one (batch, kv head, split): its p.row_tiles row groups walk the same keys. Workgroups go
    // to the eight XCDs round-robin by number, so the groups of a unit get numbers that are equal mod 8.
    const int RT = p.row_tiles;
    int unit, rt;
    {
        const int id = blockIdx.x, units = gridDim.x / RT, full = units / 8 * 8;
        if (id < full * RT) {
            const int oct = id / (8 * RT), r = id - oct * 8 * RT;
            unit = oct * 8 + (r & 7);
            rt = r >> 3;
        } else {
            const int r = id - full * RT;
            unit = full + r / RT;
            rt = r % RT;
        }
    }
    rt = RT - 1 - rt;
    const int split = unit % p.n_splits;
    unit /= p.n_splits;
    const int g = unit % p.Hkv, b = unit / p.Hkv;
    ssa_rows_pass<DQK, DV, ALIAS, NT, EXACT, MB>(p, smem, b, g, rt, split, p.n_splits);
}

// Merge of the key splits of one query row that ssa_rows_kernel left (log-sum-exp rule, fixed order), of a decode
// or (EXT) an extend:
// 128 columns a workgroup, 32 threads of four columns each, times eight groups of splits that are added in LDS at the
// end (a single chain over 64 splits took 23 us for 64 queries; whole rows a workgroup left three quarters of the
// chip idle for them: one sequence, window 8192, decode 17.4 us, now 16.9). With separate values, a result that holds a NaN or an
// infinity is computed again in fp32 (decode, see above).
template <int DQK, int DV, bool ALIAS, bool EXT>
__global__ __launch_bounds__(256) void ssa_rows_merge_kernel(const FwdParams p)
{
    constexpr int TC = 32, NG = 8;
    __shared__ f32x4 s_acc[NG][TC];
    __shared__ float s_w[64];
    __shared__ int s_odd;
    const int64_t h = blockIdx.x / (DV / 128);
    const int tc = threadIdx.x % TC, grp = threadIdx.x / TC, n = p.n_splits, col = (int)(blockIdx.x % (DV / 128)) * 128 + tc * 4;
    const float *ml = p.part_ml + h * n * 4;
    if (threadIdx.x < 64) {                        // one wave; n <= 64
        const int s = threadIdx.x;
        const float m = s < n ? ml[4 * s] : LOZA_NEG_INF, l = s < n ? ml[4 * s + 1] : 0.f;
        float mx = m;
        for (int d = 32; d > 0; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
        const float w = m == LOZA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(m - mx);
        float ls = w * l;
        for (int d = 32; d > 0; d >>= 1) ls += __shfl_xor(ls, d, 64);
        s_w[s] = ls > 0.f ? w / ls : 0.f;          // (an empty cache gives 0)
        if (s == 0) s_odd = 0;
        if (s == 0 && col == 0) {
            int64_t at = h;
            if constexpr (EXT) {                   // row (b, qi, head) of out, [b, head, qi] of lse
                const int64_t bq = h / p.Hq, b = bq / p.q_len;
                at = (b * p.Hq + (h - bq * p.Hq)) * p.q_len + (bq - b * p.q_len);
            }
            p.lse[at] = (mx + __builtin_amdgcn_logf(ls)) * 0.69314718055994530942f;
        }
    }
    __syncthreads();
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float *po = p.part_o + h * n * DV + col;
#pragma unroll 4
    for (int s = grp; s < n; s += NG) acc += s_w[s] * *(const f32x4 *)(po + (int64_t)s * DV);
    s_acc[grp][tc] = acc;
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int q = 1; q < NG; ++q) acc += s_acc[q][tc];
    if constexpr (!ALIAS && !EXT) {
        if ((acc[0] * 0.f + acc[1] * 0.f) + (acc[2] * 0.f + acc[3] * 0.f) != 0.f) s_odd = 1;
        lds_barrier();
        if (*(volatile int *)&s_odd) {
            decode_row_direct<DQK, DV>(p, h, decode_keys(p, h));
            return;
        }
    }
    u32x2 w2;
    w2[0] = pack_bf16(acc[0], acc[1]);
    w2[1] = pack_bf16(acc[2], acc[3]);
    *(u32x2 *)(p.out + h * DV + col) = w2;
}

template <int DQK, int DV, bool ALIAS, bool NT, bool EXACT, int MB = 1>
static hipError_t launch_rows_t(const FwdParams &p, hipStream_t stream)
{
    using C = RowsCfg<DQK, DV, ALIAS>;
    constexpr auto kern = ssa_rows_kernel<DQK, DV, ALIAS, NT, EXACT, MB>;
    hipError_t e = allow_lds<kern>(C::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int64_t blocks = (int64_t)p.n_splits * p.row_tiles * p.Hkv * p.B;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), C::LDS_BYTES, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess || p.n_splits == 1) return e;
    hipLaunchKernelGGL((ssa_rows_merge_kernel<DQK, DV, ALIAS, !EXACT>), dim3((unsigned)((int64_t)p.B * p.q_len * p.Hq * (DV / 128))), dim3(256), 0, stream, p);
    return hipGetLastError();
}

// One group of rows per key head reads every key row once: its copies carry the non-temporal hint (d = 128, 4
// query heads on a key head, 16 sequences, window 4096: 48.5 against 57.0 us). Several groups share the rows
// through L2 and keep the default policy (with the hint, 43 sequences of the paper's pattern: 33.3 against 30.9 us).
template <int DQK, int DV, bool ALIAS>
static hipError_t launch_rows_d(FwdParams p, bool decode, hipStream_t stream)
{
    const int64_t rows = (p.seqlens ? (int64_t)p.q_len : p.S) * p.G;
    p.row_tiles = (int)((rows + 15) / 16);
    // More than one round of the chip, but one in pairs, width 128: 32 rows a workgroup, whose every fragment from LDS feeds two
    // matrix instructions (a step 0.78 us instead of 0.68, in one round instead of two: 8 key heads, 200 tokens of window 4096 77.7 -> 55.3 us, 16 x 16 of 1 + 7 blocks 27.9 -> 19.9; up to one
    // round 41 against 55). The wide shape gains nothing by it (256 groups 148 against 322 with half the workgroups):
    // a wave's own instructions bound it there.
    if constexpr (DQK == 128) {
        const int64_t heads = (int64_t)p.Hkv * p.B;
        if (!decode && p.row_tiles * heads > 256 && (rows + 31) / 32 * heads <= 256 && p.n_splits == 1) {
            p.row_tiles = (int)((rows + 31) / 32);
            return launch_rows_t<DQK, DV, ALIAS, false, false, 2>(p, stream);
        }
    }
    if (decode) return p.row_tiles == 1 ? launch_rows_t<DQK, DV, ALIAS, true, true>(p, stream) : launch_rows_t<DQK, DV, ALIAS, false, true>(p, stream);
    return p.row_tiles == 1 ? launch_rows_t<DQK, DV, ALIAS, true, false>(p, stream) : launch_rows_t<DQK, DV, ALIAS, false, false>(p, stream);
}

hipError_t launch_rows_bf16(const FwdParams &p, int d_qk, int d_v, bool alias, bool decode, hipStream_t stream)
{
    if (d_qk == 576 && d_v == 512 && alias) return launch_rows_d<576, 512, true>(p, decode, stream);
    if (d_qk == 128 && d_v == 128) return alias ? launch_rows_d<128, 128, true>(p, decode, stream) : launch_rows_d<128, 128, false>(p, decode, stream);
    return hipErrorInvalidValue;
}

}  // namespace loza
