// A decode query computed without matrix instructions, for the kernels that finish one (gfx950).
#ifndef LOZA_SSA_DIRECT_H
#define LOZA_SSA_DIRECT_H

#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

// The live keys of decode query h = b * Hq + query head: [0, se) and [wb, length).
struct DecodeKeys {
    int b, g;
    int64_t se, wb, n_live;
};

static __device__ __forceinline__ DecodeKeys decode_keys(const FwdParams &p, int64_t h)
{
    DecodeKeys k;
    k.b = (int)(h / p.Hq);
    k.g = (int)(h - (int64_t)k.b * p.Hq) / p.G;
    const int64_t L = (int64_t)p.seqlens[k.b] < p.S ? (int64_t)p.seqlens[k.b] : p.S;
    k.se = p.n_sink < L ? p.n_sink : L;
    k.wb = L > 0 ? window_begin_of((int)(L - 1), p.window, p.block) : 0;
    if (k.wb < k.se) k.wb = k.se;
    k.n_live = k.se + (L - k.wb);
    return k;
}

// One decode query computed from the cache rows themselves: scores, softmax and weighted sum in fp32
// (no rounding of the weights). All threads of the workgroup call it together; one per four output columns
// works. The live keys are walked twice, in chunks of kDirectKeys: once for the maximum of the
// scores, once for the weights and the weighted sum (a query whose keys fit one chunk keeps its
// scores between the two). n_live >= 1.
template <int DQK, int DV>
static __device__ void decode_row_direct(const FwdParams &p, int64_t h, const DecodeKeys &keys)
{
    constexpr int NT = DV / 4;
    __shared__ float s_w[kDirectKeys];
    __shared__ __attribute__((aligned(16))) float s_q[DQK];
    __shared__ float s_m[NT];
    const int tid = threadIdx.x, c = tid * 4, b = keys.b, g = keys.g;
    const int64_t se = keys.se, wb = keys.wb, n_live = keys.n_live;
    const bool works = tid < NT;
    const int64_t k_step = (int64_t)p.Hkv * DQK;
    const bool alias = (p.v == p.k);
    const int64_t v_step = (int64_t)p.Hkv * (alias ? DQK : DV);
    const bool paged = p.block_table != nullptr;
    const int64_t seq_row0 = paged ? 0 : (int64_t)b * p.S;
    const uint16_t *kb = p.k + (seq_row0 * p.Hkv + g) * DQK;
    const uint16_t *vb = p.v + (seq_row0 * p.Hkv + g) * (alias ? DQK : DV);
    // cache row of the t-th live key (through the block table of a paged cache)
    auto key_of = [&](int64_t t) {
        const int64_t j = t < se ? t : wb + (t - se);
        if (!paged) return j;
        int pid = p.block_table[(int64_t)b * p.max_pages + (j >> p.page_shift)];
        pid = pid < 0 ? 0 : (pid < p.num_pages ? pid : p.num_pages - 1);
        return ((int64_t)pid << p.page_shift) + (j & ((1 << p.page_shift) - 1));
    };
    auto lo16 = [](uint32_t w) { return __builtin_bit_cast(float, w << 16); };
    auto hi16 = [](uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); };
    const uint16_t *q = p.q + h * DQK;
    for (int e = tid; works && e < DQK; e += NT) s_q[e] = __builtin_bit_cast(float, (uint32_t)q[e] << 16);
    __syncthreads();
    // scale * log2(e) * q . k of the t-th live key
    auto score = [&](int64_t t) {
        const u32x4 *kr = (const u32x4 *)(kb + key_of(t) * k_step);
        float dot = 0.f;
#pragma unroll 2
        for (int c8 = 0; c8 < DQK / 8; ++c8) {
            const u32x4 w = kr[c8];
            const float4 qa = *(const float4 *)(s_q + 8 * c8), qb = *(const float4 *)(s_q + 8 * c8 + 4);
            dot = __builtin_fmaf(qa.x, lo16(w[0]), dot);
            dot = __builtin_fmaf(qa.y, hi16(w[0]), dot);
            dot = __builtin_fmaf(qa.z, lo16(w[1]), dot);
            dot = __builtin_fmaf(qa.w, hi16(w[1]), dot);
            dot = __builtin_fmaf(qb.x, lo16(w[2]), dot);
            dot = __builtin_fmaf(qb.y, hi16(w[2]), dot);
            dot = __builtin_fmaf(qb.z, lo16(w[3]), dot);
            dot = __builtin_fmaf(qb.w, hi16(w[3]), dot);
        }
        return dot * p.scale_log2;
    };
    const bool one_chunk = n_live <= kDirectKeys;
    float m = LOZA_NEG_INF;
    for (int64_t t = tid; works && t < n_live; t += NT) {
        const float sc = score(t);
        if (one_chunk) s_w[t] = sc;
        m = fmaxf(m, sc);
    }
    if (works) s_m[tid] = m;
    __syncthreads();
    for (int t = 0; t < NT; ++t) m = fmaxf(m, s_m[t]);
    float l = 0.f;
    float4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t c0 = 0; c0 < n_live; c0 += kDirectKeys) {
        const int cnt = (int)(n_live - c0 < kDirectKeys ? n_live - c0 : kDirectKeys);
        for (int t = tid; works && t < cnt; t += NT) s_w[t] = __builtin_amdgcn_exp2f((one_chunk ? s_w[t] : score(c0 + t)) - m);
        __syncthreads();
        for (int t = 0; works && t < cnt; ++t) {
            const float w = s_w[t];
            const u32x2 vr = *(const u32x2 *)(vb + key_of(c0 + t) * v_step + c);
            l += w;
            acc.x = __builtin_fmaf(w, lo16(vr[0]), acc.x);
            acc.y = __builtin_fmaf(w, hi16(vr[0]), acc.y);
            acc.z = __builtin_fmaf(w, lo16(vr[1]), acc.z);
            acc.w = __builtin_fmaf(w, hi16(vr[1]), acc.w);
        }
        __syncthreads();
    }
    if (!works) return;
    const float inv = 1.0f / l;
    u32x2 w2;
    w2[0] = pack_bf16(acc.x * inv, acc.y * inv);
    w2[1] = pack_bf16(acc.z * inv, acc.w * inv);
    *(u32x2 *)(p.out + h * DV + c) = w2;
    if (tid == 0) p.lse[h] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
}

}  // namespace loza
#endif
