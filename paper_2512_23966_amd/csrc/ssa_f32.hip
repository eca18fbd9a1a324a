// fp32 streaming sparse attention for gfx950: fp32 in, fp32 arithmetic, fp32 out.
//
// O* = softmax(scale * Q K*^T) V* over live(i) = { j <= i : j < n_sink or i - j < window }
// (paper: Architecture section, Eq. 2 / Eq. 4).  This is the small, exact-arithmetic twin of the
// bf16 kernels, forward (prefill and decode) and backward.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ssa_device.h"
#include "ssa_kernels.h"

namespace loza {

constexpr int F32_MAX_D = 256;
constexpr int F32_WAVES = 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load, 4-byte aligned

// Forward. A workgroup owns 16 query rows (position, head) of one key/value head; its NW waves share the
// keys in tiles of 16 (tile number mod NW), each with its own softmax state and accumulators, and the
// partial results meet in LDS once. Both products run on the fp32 matrix instruction (16x16x4, full fp32):
// S^T[16 keys][16 rows] = K Q^T leaves lane (j, n) with row n's scores of keys 4j .. 4j + 3, and step i of
// O^T += V^T P^T contracts keys 4j + i over j, so the probabilities are used where they are. The order of a
// contraction and of the output columns is free, so every global load is 16 bytes a lane: feature
// 16 kk + 4 j + e takes part in step e, column 64 d + 4 m + e is row m of block e.
// What bounds it at these sizes is latency (1024 rows of 320 keys of width 64 are 64 workgroups of three
// tiles a wave): one wave per row, one key per lane with strided 4-byte loads and a serial sum over the keys
// took 80 us, this 9 (in a graph, without the host's share: 9.95 with a branch around every load and the maximum
// exchanged in every tile, now 9.4; 2,048 rows of 4 heads of width 128, window 512: 45.7 and 40).
// The online softmax takes each row's own running maximum, and a tile without a live key of a
// row leaves that row's state exactly as it was: a row's result does not depend on the rows it shares a
// workgroup with, and a decode gives the bits of the prefill's last row. (The matrix instruction multiplies
// every row's weight, 0 where the key is dead, with every value of the tile: a wave whose sums are not all
// finite walks its keys again and adds each to the rows that see it.)
// ND: blocks of 64 features and columns (the widths are cut to d_qk and d_v inside). VEC: widths that are
// multiples of 4 (rows 16-byte aligned); otherwise the 16-byte loads are aligned to 4 bytes, and at the end of a
// row four scalar ones.
template <int ND>
struct F32RowsCfg {
    static constexpr int NW = ND <= 2 ? 8 : 4;         // (wider rows need the registers)
    static constexpr int OROW = ND * 64 + 4;           // floats per row of a wave's partial output
    static constexpr int LDS_BYTES = (NW * 16 * OROW + NW * 16 * 2) * 4;
    static_assert(LDS_BYTES <= 160 * 1024, "does not fit the 160 KB LDS");
};

// DX: d_qk = d_v = DX (64, 96, 128), known to the compiler: no lane asks whether its columns exist, and no step of
// the scores is taken of nothing; 0: any widths.
template <int ND, bool VEC, int DX>
__global__ __launch_bounds__(64 * F32RowsCfg<ND>::NW) void ssa_rows_f32_kernel(const F32Params p, const int row_tiles)
{
    using C = F32RowsCfg<ND>;
    static_assert(DX == 0 || (VEC && DX <= 64 * ND), "widths");
    const int d_qk = DX ? DX : p.d_qk, d_v = DX ? DX : p.d_v;
    constexpr int KQ = DX ? DX / 16 : ND * 4;               // steps of 16 features
    constexpr int NW = C::NW, N = 16, OROW = C::OROW;
    extern __shared__ __attribute__((aligned(16))) float smem_f[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n16 = lane & 15, j4 = lane >> 4;
    const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (id >= (int64_t)row_tiles * p.Hkv * p.B) return;
    int rt, g, b;
    if (id <= 0x7fffffff) {                                  // (a 64-bit division takes more than a hundred instructions)
        const int bg = (int)id / row_tiles;
        rt = (int)id - bg * row_tiles;
        b = bg / p.Hkv;
        g = bg - b * p.Hkv;
    } else {
        const int64_t bg = id / row_tiles;
        rt = (int)(id - bg * row_tiles);
        b = (int)(bg / p.Hkv);
        g = (int)(bg - (int64_t)b * p.Hkv);
    }
    const int G = p.Hq / p.Hkv;
    const bool decode = p.seqlens != nullptr;
    // valid keys (a length beyond the cache is cut to it); queries are its last (decode) or all positions
    const int64_t L = decode ? ((int64_t)p.seqlens[b] < p.S ? (int64_t)p.seqlens[b] : p.S) : p.S;
    const int64_t Sq = decode ? 1 : p.S, pos0 = L - Sq, R = Sq * G, r0 = (int64_t)rt * 16;
    const int n_sink = p.n_sink, block = p.block;
    auto window_begin = [&](int i) {
        const int qblk = block == 1 ? i : i / block;
        return p.window > qblk ? 0 : (qblk - p.window + 1) * block;
    };
    const int i_min = (int)(pos0 + row_position(r0, G)), i_max = (int)(pos0 + row_position(r0 + 15 < R ? r0 + 15 : R - 1, G));

    // elements c .. c + 3 of a row of d, 0 past its end; the wave's lanes ask for [base, base + span) together
    auto load4 = [&](const float *row, int c, int d, int base, int span) -> f32x4 {
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DX > 0) {
            if (base + span <= DX) {
                x = *(const f32x4 *)(row + c);
            } else {                                         // (96: half of the second block's lanes; the others load what they drop)
                const f32x4 y = *(const f32x4 *)(row + (c < DX ? c : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = c < DX ? y[e] : 0.f;
            }
        } else if constexpr (VEC) {
            if (c < d) x = *(const f32x4 *)(row + c);
        } else if (base + span <= d) {
            x = *(const f32x4_dword *)(row + c);
        } else {
            // (a lane past the end loads the row's start and drops it: no branch around every load)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = row[c + e < d ? c + e : 0];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = c + e < d ? x[e] : 0.f;
        }
        return x;
    };

    // this lane's query row (its matrix-core operand), and the row's window
    const int64_t my_row = r0 + n16, row_c = my_row < R ? my_row : R - 1, qi = row_position(row_c, G);
    const int i_row = (int)(pos0 + qi), w_lo_row = window_begin(i_row < 0 ? 0 : i_row);
    const int64_t q_row = ((int64_t)b * Sq + qi) * p.Hq + (int64_t)g * G + (row_c - qi * G);
    f32x4 qf[KQ];
#pragma unroll
    for (int kk = 0; kk < KQ; ++kk) qf[kk] = load4(p.q + q_row * d_qk, kk * 16 + j4 * 4, d_qk, kk * 16, 16);

    // live key tiles: [0, nA) and [wt0, wt1]; this wave takes those whose number is `wave` mod NW
    const int win_begin = window_begin(i_min < 0 ? 0 : i_min);
    const int sink_end = n_sink < i_max + 1 ? n_sink : i_max + 1;
    int nA = (sink_end + N - 1) / N;
    int wt0 = win_begin / N;
    const int wt1 = i_max < 0 ? -1 : i_max / N;                 // (an empty cache has no tile)
    if (i_max < 0) nA = 0;
    if (wt0 < nA) wt0 = nA;
    auto next_tile = [&](int t) {                               // first tile of this wave at or after t
        t += (wave - t % NW + NW) % NW;
        if (t >= nA && t < wt0) { t = wt0; t += (wave - t % NW + NW) % NW; }
        return t;
    };
    const float *kb = p.k + ((int64_t)b * p.S * p.Hkv + g) * p.k_row;
    const float *vb = p.v + ((int64_t)b * p.S * p.Hkv + g) * p.v_row;
    const int64_t kstep = (int64_t)p.Hkv * p.k_row, vstep = (int64_t)p.Hkv * p.v_row;
    // a key that no row of this group sees is never read: a live one is loaded in its place (and masked)
    auto live_key = [&](int j) {
        if (j >= n_sink && j < win_begin) j = win_begin;
        return j < i_max ? j : i_max;
    };
    f32x4 kf[KQ];
    auto load_keys = [&](int t) {
        const float *kr = kb + (int64_t)live_key(t * N + n16) * kstep;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) kf[kk] = load4(kr, kk * 16 + j4 * 4, d_qk, kk * 16, 16);
    };

    f32x4 o[ND][4];
    float m, l;
    auto walk = [&](auto by_key_c) {
        constexpr bool BY_KEY = decltype(by_key_c)::value;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[d][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        m = -INFINITY;
        l = 0.f;
        int t = next_tile(0);
        if (t <= wt1) load_keys(t);
        while (t <= wt1) {
            f32x4 vf[4][ND];                                    // values of keys 4 j4 + i
            if constexpr (!BY_KEY) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float *vr = vb + (int64_t)live_key(t * N + 4 * j4 + i) * vstep;
#pragma unroll
                    for (int d = 0; d < ND; ++d) vf[i][d] = load4(vr, d * 64 + n16 * 4, d_v, d * 64, 64);
                }
            }
            f32x4 s4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s4[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KQ; ++kk)
#pragma unroll
                for (int e = 0; e < 4; ++e) s4[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kk][e], qf[kk][e], s4[e], 0, 0, 0);
            const int t_next = next_tile(t + 1);
            if (t_next <= wt1) load_keys(t_next);
            f32x4 s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            float cm = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = t * N + 4 * j4 + i;
                const bool ok = (j <= i_row) & ((j < n_sink) | (j >= w_lo_row));
                s[i] = ok ? s[i] * p.scale : -INFINITY;
                cm = fmaxf(cm, s[i]);
            }
            // (each row's running maximum, whatever the rows beside it do; past the first tiles it seldom moves. A
            // reference that may be exceeded by e^8 and a shorter exponential were another 4 % faster, and 0.4 % less exact.
            // With the branches of any widths around every load, asking first costs more than the exchange: 1,548 rows
            // of width 32, 27.2 us and 26.6.)
            if (DX == 0 || __any(cm > m)) {
                cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
                cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
                const float alpha = cm > m ? expf(m - cm) : 1.f;
                m = fmaxf(m, cm);
                l *= alpha;
#pragma unroll
                for (int d = 0; d < ND; ++d)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[d][e] *= alpha;
            }
            const float m_use = m == -INFINITY ? 0.f : m;           // a row without a live key so far
            float ps = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[i] = s[i] == -INFINITY ? 0.f : expf(s[i] - m_use);
                ps += s[i];
            }
            l += ps;
            if constexpr (!BY_KEY) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int d = 0; d < ND; ++d)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[d][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][d][e], s[i], o[d][e], 0, 0, 0);
            }
            if constexpr (BY_KEY) {
#pragma unroll 1
                for (int jq = 0; jq < 4; ++jq)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int j = t * N + 4 * jq + i;
                        const float w = __shfl(s[i], jq * 16 + n16, 64);
                        if (!((j <= i_row) & ((j < n_sink) | (j >= w_lo_row)))) continue;
                        const float *vr = vb + (int64_t)live_key(j) * vstep;
#pragma unroll
                        for (int d = 0; d < ND; ++d)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {        // columns of o[d][.][r]
                                const f32x4 x = load4(vr, d * 64 + j4 * 16 + r * 4, d_v, d * 64, 64);
#pragma unroll
                                for (int e = 0; e < 4; ++e) o[d][e][r] = fmaf(w, x[e], o[d][e][r]);
                            }
                    }
            }
            t = t_next;
        }
    };
    walk(std::false_type{});
    {
        float odd[4] = {0.f, 0.f, 0.f, 0.f};                    // 0 if every accumulator is finite, else NaN
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) odd[i] = fmaf(o[d][e][i], 0.f, odd[i]);
        if (__any((odd[0] + odd[1]) + (odd[2] + odd[3]) != 0.f)) walk(std::true_type{});
    }

    // ---- the waves' partial results meet in LDS ---------------------------------------------------------
    float *ml = smem_f + NW * 16 * OROW;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (j4 == 0) {
        ml[(wave * 16 + n16) * 2] = m;
        ml[(wave * 16 + n16) * 2 + 1] = l;
    }
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // lane (j4, n16): columns d * 64 + 16 j4 + 4 i + e of row n16
            const f32x4 w = {o[d][0][i], o[d][1][i], o[d][2][i], o[d][3][i]};
            *(f32x4 *)(smem_f + (wave * 16 + n16) * OROW + d * 64 + j4 * 16 + i * 4) = w;
        }
    __syncthreads();
    for (int x = threadIdx.x; x < 16 * ND * 16; x += 64 * NW) {
        const int rr = x / (ND * 16), c = (x % (ND * 16)) * 4;
        const int64_t row = r0 + rr;
        if (row >= R || c >= d_v) continue;
        float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, ml[(w * 16 + rr) * 2]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = ml[(w * 16 + rr) * 2], a = mw == -INFINITY ? 0.f : expf(mw - m_all);
            l_all += a * ml[(w * 16 + rr) * 2 + 1];
            acc += a * *(const f32x4 *)(smem_f + (w * 16 + rr) * OROW + c);
        }
        // (an empty cache gives 0 and -inf; live keys whose scores are all -inf have no softmax)
        const float inv = L > 0 ? 1.0f / l_all : 0.f;
        const int64_t i = row_position(row, G);
        const int64_t h = (int64_t)g * G + (row - i * G);
        float *op = p.out + (((int64_t)b * Sq + i) * p.Hq + h) * d_v + c;
        if constexpr (VEC) {
            *(f32x4 *)op = acc * inv;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < d_v) op[e] = acc[e] * inv;
        }
        if (c == 0) p.lse[((int64_t)b * p.Hq + h) * Sq + i] = L > 0 && l_all == 0.f ? __builtin_nanf("") : m_all + logf(l_all);
    }
}

template <int ND, bool VEC, int DX = 0>
static hipError_t launch_rows_f32_t(const F32Params &p, hipStream_t stream)
{
    using C = F32RowsCfg<ND>;
    constexpr auto kern = ssa_rows_f32_kernel<ND, VEC, DX>;
    hipError_t e = allow_lds<kern>(C::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int64_t rows = (p.seqlens ? 1 : p.S) * (p.Hq / p.Hkv), row_tiles = (rows + 15) / 16;
    // (a grid row holds fewer than 2^32 threads)
    const int64_t blocks = row_tiles * p.Hkv * p.B, gx = blocks < (1 << 22) ? blocks : (1 << 22), gy = (blocks + gx - 1) / gx;
    hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)gy), dim3(64 * C::NW), C::LDS_BYTES, stream, p, (int)row_tiles);
    return hipGetLastError();
}

template <bool VEC>
static hipError_t launch_rows_f32(const F32Params &p, hipStream_t stream)
{
    const int d = p.d_qk > p.d_v ? p.d_qk : p.d_v;
    // The usual head widths are known to the compiler: without a branch around every load 1,024 rows of one head of width
    // 64 take 9.4 us instead of 9.95, 2,048 rows of 4 heads of width 128 40 instead of 45.7, 266 rows of width 96 11.5
    // instead of 12.9. Any other width would gain by a kernel of its own likewise; these three are what is in use.
    if constexpr (VEC) {
        if (p.d_qk == p.d_v && d == 64) return launch_rows_f32_t<1, true, 64>(p, stream);
        if (p.d_qk == p.d_v && d == 96) return launch_rows_f32_t<2, true, 96>(p, stream);
        if (p.d_qk == p.d_v && d == 128) return launch_rows_f32_t<2, true, 128>(p, stream);
    }
    if (d <= 64) return launch_rows_f32_t<1, VEC>(p, stream);
    if (d <= 128) return launch_rows_f32_t<2, VEC>(p, stream);
    if (d <= 192) return launch_rows_f32_t<3, VEC>(p, stream);
    return launch_rows_f32_t<4, VEC>(p, stream);
}

hipError_t launch_prefill_f32(const F32Params &p, hipStream_t stream)
{
    // (base pointers are 16-byte aligned; rows of a multiple of four floats then are, too)
    const bool vec = p.d_qk % 4 == 0 && p.d_v % 4 == 0;
    return vec ? launch_rows_f32<true>(p, stream) : launch_rows_f32<false>(p, stream);
}

// ---- fp32 backward (the small, exact-arithmetic twin of ssa_bwd.hip) --------------------------------
// With p_ij = exp(scale q_i.k_j - lse_i) over live pairs, D_i = dO_i . O_i, dP_ij = dO_i . v_j and
// dS_ij = p_ij (dP_ij - D_i):   dQ_i = scale sum_j dS_ij k_j,  dK_j = scale sum_i dS_ij q_i,
// dV_j = sum_i p_ij dO_i   (the derivative of the paper's Eq. 4; Architecture section, Training).
// Two kernels, no atomics: one wavefront per query row walks that row's live keys (dQ); one wavefront
// per key walks the query rows that see it (dK, dV), 64 at a time, one per lane for the scalars and
// one gradient column per lane for the sums.

// per-lane dot product of two rows of n floats
static __device__ __forceinline__ float dot_rows(const float *a, const float *b, int n)
{
    float d = 0.f;
    for (int c = 0; c < n; ++c) d = fmaf(a[c], b[c], d);
    return d;
}

__global__ __launch_bounds__(64 * F32_WAVES) void ssa_backward_f32_dq_kernel(const F32BwdParams p)
{
    __shared__ float s_q[F32_WAVES][F32_MAX_D], s_do[F32_WAVES][F32_MAX_D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t n_rows = (int64_t)p.B * p.S * p.Hq;
    const int64_t r = (int64_t)blockIdx.x * F32_WAVES + wave;
    if (r >= n_rows) return;  // whole wavefront leaves together; no block-wide barrier is used
    const int h = (int)(r % p.Hq);
    const int64_t bi = r / p.Hq;
    const int i = (int)(bi % p.S);
    const int64_t b = bi / p.S;
    const int g = h / (p.Hq / p.Hkv);

    float dpart = 0.f;  // D = dO . O
    for (int c = lane; c < p.d_qk; c += 64) s_q[wave][c] = p.q[r * p.d_qk + c];
    for (int c = lane; c < p.d_v; c += 64) {
        const float d = p.dout[r * p.d_v + c];
        s_do[wave][c] = d;
        dpart = fmaf(d, p.out[r * p.d_v + c], dpart);
    }
    for (int off = 32; off > 0; off >>= 1) dpart += __shfl_xor(dpart, off, 64);
    const float D = dpart;
    const float lse = p.lse[((int64_t)b * p.Hq + h) * p.S + i];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

    const int se = p.n_sink < i + 1 ? p.n_sink : i + 1;
    const int qblk = i / p.block;
    int wb = p.window > qblk ? 0 : (qblk - p.window + 1) * p.block;
    if (wb < se) wb = se;
    const int n_live = se + (i - wb + 1);
    const float *kb = p.k + ((int64_t)b * p.S * p.Hkv + g) * p.k_row;
    const float *vb = p.v + ((int64_t)b * p.S * p.Hkv + g) * p.v_row;
    const int64_t kstep = (int64_t)p.Hkv * p.k_row, vstep = (int64_t)p.Hkv * p.v_row;

    float acc[F32_MAX_D / 64];
#pragma unroll
    for (int c = 0; c < F32_MAX_D / 64; ++c) acc[c] = 0.f;
    for (int u0 = 0; u0 < n_live; u0 += 64) {
        const int u = u0 + lane;
        const bool have = u < n_live;
        const int j = have ? (u < se ? u : wb + (u - se)) : 0;
        float ds = 0.f;
        if (have) {
            const float s = dot_rows(s_q[wave], kb + (int64_t)j * kstep, p.d_qk) * p.scale;
            const float pj = expf(s - lse);
            const float dp = dot_rows(s_do[wave], vb + (int64_t)j * vstep, p.d_v);
            ds = pj * (dp - D);
        }
        const int cnt = n_live - u0 < 64 ? n_live - u0 : 64;
        for (int jj = 0; jj < cnt; ++jj) {
            const float w = __shfl(ds, jj, 64);
            const float *kr = kb + (int64_t)__shfl(j, jj, 64) * kstep;
#pragma unroll
            for (int c = 0; c < F32_MAX_D / 64; ++c) {
                const int col = c * 64 + lane;
                if (col < p.d_qk) acc[c] = fmaf(w, kr[col], acc[c]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < F32_MAX_D / 64; ++c) {
        const int col = c * 64 + lane;
        if (col < p.d_qk) p.dq[r * p.d_qk + col] = acc[c] * p.scale;
    }
}

__global__ __launch_bounds__(64 * F32_WAVES) void ssa_backward_f32_dkv_kernel(const F32BwdParams p)
{
    __shared__ float s_k[F32_WAVES][F32_MAX_D], s_v[F32_WAVES][F32_MAX_D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t n_keys = (int64_t)p.B * p.S * p.Hkv;
    const int64_t kr_idx = (int64_t)blockIdx.x * F32_WAVES + wave;  // flat (b, j, g)
    if (kr_idx >= n_keys) return;
    const int g = (int)(kr_idx % p.Hkv);
    const int64_t bj = kr_idx / p.Hkv;
    const int j = (int)(bj % p.S);
    const int64_t b = bj / p.S;
    const int G = p.Hq / p.Hkv;

    for (int c = lane; c < p.d_qk; c += 64) s_k[wave][c] = p.k[kr_idx * p.k_row + c];
    for (int c = lane; c < p.d_v; c += 64) s_v[wave][c] = p.v[kr_idx * p.v_row + c];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

    // the positions that see key j: every later one for a sink key, else those whose window still
    // holds it: i / block - window + 1 <= j / block
    int64_t i_last = p.S - 1;
    if (j >= p.n_sink) {
        const int64_t jb = j / p.block, last_blk = (p.S - 1) / p.block;
        if (jb + p.window - 1 < last_blk) i_last = (jb + p.window) * p.block - 1;  // (< S: no overflow)
    }
    const int64_t n_rows = (i_last - j + 1) * G;  // rows (i, head of the group), position-major

    float acc_k[F32_MAX_D / 64], acc_v[F32_MAX_D / 64];
#pragma unroll
    for (int c = 0; c < F32_MAX_D / 64; ++c) { acc_k[c] = 0.f; acc_v[c] = 0.f; }
    for (int64_t u0 = 0; u0 < n_rows; u0 += 64) {
        const int64_t u = u0 + lane;
        const bool have = u < n_rows;
        float pj = 0.f, ds = 0.f;
        if (have) {
            const int64_t i = j + u / G;
            const int h = g * G + (int)(u % G);
            const int64_t row = ((int64_t)b * p.S + i) * p.Hq + h;  // flat (b, i, h)
            const float *qr = p.q + row * p.d_qk, *dor = p.dout + row * p.d_v;
            const float s = dot_rows(qr, s_k[wave], p.d_qk) * p.scale;
            pj = expf(s - p.lse[((int64_t)b * p.Hq + h) * p.S + i]);
            const float dp = dot_rows(dor, s_v[wave], p.d_v);
            const float D = dot_rows(dor, p.out + row * p.d_v, p.d_v);
            ds = pj * (dp - D);
        }
        const int cnt = n_rows - u0 < 64 ? (int)(n_rows - u0) : 64;
        for (int jj = 0; jj < cnt; ++jj) {
            const float wk = __shfl(ds, jj, 64), wv = __shfl(pj, jj, 64);
            const int64_t uu = u0 + jj;
            const int64_t rr = ((int64_t)b * p.S + j + uu / G) * p.Hq + g * G + (int)(uu % G);
            const float *qr = p.q + rr * p.d_qk, *dor = p.dout + rr * p.d_v;
#pragma unroll
            for (int c = 0; c < F32_MAX_D / 64; ++c) {
                const int col = c * 64 + lane;
                if (col < p.d_qk) acc_k[c] = fmaf(wk, qr[col], acc_k[c]);
                if (col < p.d_v) acc_v[c] = fmaf(wv, dor[col], acc_v[c]);
            }
        }
    }
    // values that are a prefix of the key rows: one tensor, one gradient (dK with dV added to its
    // first d_v columns), and no dv is written
#pragma unroll
    for (int c = 0; c < F32_MAX_D / 64; ++c) {
        const int col = c * 64 + lane;
        if (p.dv == nullptr) {
            if (col < p.d_qk) p.dk[kr_idx * p.d_qk + col] = acc_k[c] * p.scale + (col < p.d_v ? acc_v[c] : 0.f);
        } else {
            if (col < p.d_qk) p.dk[kr_idx * p.d_qk + col] = acc_k[c] * p.scale;
            if (col < p.d_v) p.dv[kr_idx * p.d_v + col] = acc_v[c];
        }
    }
}

hipError_t launch_backward_f32(const F32BwdParams &p, hipStream_t stream)
{
    const int64_t n_rows = (int64_t)p.B * p.S * p.Hq, n_keys = (int64_t)p.B * p.S * p.Hkv;
    hipLaunchKernelGGL(ssa_backward_f32_dq_kernel, dim3((unsigned)((n_rows + F32_WAVES - 1) / F32_WAVES)), dim3(64 * F32_WAVES), 0,
                       stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ssa_backward_f32_dkv_kernel, dim3((unsigned)((n_keys + F32_WAVES - 1) / F32_WAVES)), dim3(64 * F32_WAVES), 0,
                       stream, p);
    return hipGetLastError();
}

}  // namespace loza
