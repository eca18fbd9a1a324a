// How the backward kernels of the wide shape bring a tile to LDS and read it (device side).
#ifndef LOZA_SSA_BWD_TILE_H
#define LOZA_SSA_BWD_TILE_H

#include "ssa_device.h"

namespace loza {

namespace {

// One global -> LDS copy instruction: 64 lanes x 16 bytes from base + off (per lane) to the 1 KB of
// LDS at lds_addr (wave-uniform, through M0). The compiler's wait counters do not see it: the tile
// loops wait for their copies themselves before the barrier that publishes a tile.
__device__ __forceinline__ void copy_1k(const char *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// The same for data that is read once: not kept in L2.
__device__ __forceinline__ void copy_1k_once(const char *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 0\n global_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// The same to lds_addr + step (a constant), of the lane's offset cut at `max`: three instructions.
template <int STEP>
__device__ __forceinline__ void copy_1k_cut(const char *base, uint32_t off, uint32_t max, uint32_t lds_addr)
{
    uint32_t tmp;
    asm volatile("s_add_u32 m0, %3, %5\n v_min_u32 %0, %1, %4\n global_load_lds_dwordx4 %0, %2"
                 : "=&v"(tmp) : "v"(off), "s"(base), "s"(lds_addr), "s"(max), "n"(STEP) : "memory", "m0", "scc");
}

// Two transposing 64-bit reads: matrix-core operand of lane (half h, n), whose eight values of the contraction are
// what the lanes' own addresses a and b say: four each.
__device__ __forceinline__ bf16x8 read_tr_pair(const char *a, const char *b)
{
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(b));
    s16x8 a8;
    a8[0] = lo[0]; a8[1] = lo[1]; a8[2] = lo[2]; a8[3] = lo[3];
    a8[4] = hi[0]; a8[5] = hi[1]; a8[6] = hi[2]; a8[7] = hi[3];
    return __builtin_bit_cast(bf16x8, a8);
}

// Matrix-core A operand [32 columns of block db][16 items of key step ks] of a tile stored
// [item][column] (padded rows of `row` bytes).
__device__ __forceinline__ bf16x8 read_transposed(const char *tile, int row, int db, int ks, int lane)
{
    const int lh = lane >> 5, s16 = lane & 15, g16 = (lane >> 4) & 1;
    const char *a = tile + (ks * 16 + lh * 8 + (s16 >> 2)) * row + (db * 32 + g16 * 16 + (s16 & 3) * 4) * 2;
    return read_tr_pair(a, a + 4 * row);
}

}  // namespace

}  // namespace loza
#endif
