// bf16 streaming sparse attention for few query rows (gfx950): decode, short extends, short prompts, and the last step
// of an extend whose keys several workgroups of the tile kernel shared. The pass over sixteen rows and the reasons for
// it are in ssa_rows.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssa_device.h"
#include "ssa_direct.h"
#include "ssa_kernels.h"
#include "ssa_rows.h"

namespace loza {

namespace {

// eight columns of a finished row
template <int DV>
__device__ __forceinline__ void rows_store(const FwdParams &p, int64_t o_row, int c, f32x4 lo, f32x4 hi)
{
    u32x4 w;
    w[0] = pack_bf16(lo[0], lo[1]);
    w[1] = pack_bf16(lo[2], lo[3]);
    w[2] = pack_bf16(hi[0], hi[1]);
    w[3] = pack_bf16(hi[2], hi[3]);
    *(u32x4 *)(p.out + o_row * DV + c) = w;
}

}  // namespace

// FINISH: the second launch of an extend whose key tiles ssa_bf16.hip's tile kernel has split: the workgroup adds
// the partial results of its 16 rows and is done, unless they must not come from once-rounded weights (a tile among
// the first positions, a pattern of few live keys, a large result): then it computes its rows from the keys, as it
// would without the first launch.
template <int DQK, int DV, bool ALIAS, bool NT, bool EXACT, bool FINISH = false>
__global__ __launch_bounds__(256) void ssa_rows_kernel(const FwdParams p)
{
    using C = RowsCfg<DQK, DV, ALIAS>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

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
    const int n_splits = FINISH ? 1 : p.n_splits;   // of this launch
    const int split = unit % n_splits;
    unit /= n_splits;
    const int g = unit % p.Hkv, b = unit / p.Hkv;
    if constexpr (FINISH) {
        constexpr int LPR = DV / 8, RPI = 64 / LPR;   // lanes per finished row (8 columns each), rows per step
        const int G = p.G;
        const int64_t L = (int64_t)p.seqlens[b] < p.S ? (int64_t)p.seqlens[b] : p.S;
        const int64_t Sq = (int64_t)p.q_len, pos0 = L - Sq, R = Sq * G, r0 = (int64_t)rt * 16;
        // (the first position of the tile of kTileRows rows these 16 were part of)
        const int i_tile = (int)(pos0 + row_position(r0 / kTileRows * kTileRows, G));
        if (!p.all_precise && i_tile >= kPrecisePositions) {
            int *s_big = (int *)(smem + C::OFF_ODD);
            if (tid == 0) *s_big = 0;
            __syncthreads();
            const int n = p.n_splits;
            f32x4 lo[4 / RPI], hi[4 / RPI];
            bool big = false;
#pragma unroll
            for (int step = 0; step < 4 / RPI; ++step) {
                const int64_t row = r0 + wave * 4 + step * RPI + lane / LPR, rc = row < R ? row : R - 1, qi = row_position(rc, G);
                const int64_t h = (int64_t)g * G + (rc - qi * G), o_row = ((int64_t)b * Sq + qi) * p.Hq + h;
                const int c = (lane % LPR) * 8;
                const float *ml = p.part_ml + o_row * n * 4, *po = p.part_o + o_row * n * DV + c;
                float m_all = LOZA_NEG_INF;
                for (int s = 0; s < n; ++s) m_all = fmaxf(m_all, ml[4 * s]);
                float den = 0.f, den_r = 0.f;
                f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
#pragma unroll 4
                for (int s = 0; s < n; ++s) {
                    const float a = ml[4 * s] == LOZA_NEG_INF ? 0.f : __builtin_amdgcn_exp2f(ml[4 * s] - m_all);
                    den += a * ml[4 * s + 1];
                    den_r += a * ml[4 * s + 2];
                    x += a * *(const f32x4 *)(po + (int64_t)s * DV);
                    y += a * *(const f32x4 *)(po + (int64_t)s * DV + 4);
                }
                const float inv = den_r > 0.f ? 1.0f / den_r : 0.f;
                lo[step] = x * inv;
                hi[step] = y * inv;
                float mx = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fmaxf(__builtin_fabsf(lo[step][e]), __builtin_fabsf(hi[step][e])));
                big = big || (mx >= kRedoMagnitude && row < R);
                if (c == 0 && row < R) p.lse[((int64_t)b * p.Hq + h) * Sq + qi] = (m_all + __builtin_amdgcn_logf(den)) * 0.69314718055994530942f;
            }
            if (__any(big) && lane == 0) *s_big = 1;
            __syncthreads();
            const bool again = *(volatile int *)s_big != 0;
            if (!again) {
#pragma unroll
                for (int step = 0; step < 4 / RPI; ++step) {
                    const int64_t row = r0 + wave * 4 + step * RPI + lane / LPR;
                    if (row >= R) continue;
                    const int64_t qi = row_position(row, G);
                    rows_store<DV>(p, ((int64_t)b * Sq + qi) * p.Hq + (int64_t)g * G + (row - qi * G), (lane % LPR) * 8, lo[step], hi[step]);
                }
                return;
            }
            // (the log-sum-exps written above arrive before those of the rows computed again)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __syncthreads();
        }
    }

    ssa_rows_pass<DQK, DV, ALIAS, NT, EXACT>(p, smem, b, g, rt, split, n_splits);
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

template <int DQK, int DV, bool ALIAS, bool NT, bool EXACT>
static hipError_t launch_rows_t(const FwdParams &p, hipStream_t stream)
{
    using C = RowsCfg<DQK, DV, ALIAS>;
    constexpr auto kern = ssa_rows_kernel<DQK, DV, ALIAS, NT, EXACT>;
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
    if (decode) return p.row_tiles == 1 ? launch_rows_t<DQK, DV, ALIAS, true, true>(p, stream) : launch_rows_t<DQK, DV, ALIAS, false, true>(p, stream);
    return p.row_tiles == 1 ? launch_rows_t<DQK, DV, ALIAS, true, false>(p, stream) : launch_rows_t<DQK, DV, ALIAS, false, false>(p, stream);
}

template <int DQK, int DV, bool ALIAS>
static hipError_t launch_finish_t(FwdParams p, hipStream_t stream)
{
    using C = RowsCfg<DQK, DV, ALIAS>;
    constexpr auto kern = ssa_rows_kernel<DQK, DV, ALIAS, false, false, true>;
    hipError_t e = allow_lds<kern>(C::LDS_BYTES);
    if (e != hipSuccess) return e;
    p.row_tiles = (int)(((int64_t)p.q_len * p.G + 15) / 16);
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)p.row_tiles * p.Hkv * p.B)), dim3(256), C::LDS_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_rows_finish_bf16(const FwdParams &p, int d_qk, int d_v, bool alias, hipStream_t stream)
{
    if (d_qk == 576 && d_v == 512 && alias) return launch_finish_t<576, 512, true>(p, stream);
    if (d_qk == 128 && d_v == 128) return alias ? launch_finish_t<128, 128, true>(p, stream) : launch_finish_t<128, 128, false>(p, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_rows_bf16(const FwdParams &p, int d_qk, int d_v, bool alias, bool decode, hipStream_t stream)
{
    if (d_qk == 576 && d_v == 512 && alias) return launch_rows_d<576, 512, true>(p, decode, stream);
    if (d_qk == 128 && d_v == 128) return alias ? launch_rows_d<128, 128, true>(p, decode, stream) : launch_rows_d<128, 128, false>(p, decode, stream);
    return hipErrorInvalidValue;
}

}  // namespace loza
