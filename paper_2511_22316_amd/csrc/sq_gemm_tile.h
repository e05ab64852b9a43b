// What the W4A4 tile kernels share: the swizzled LDS tile of packed codes and the order of the tiles.
#pragma once

#include "sq_common.h"

namespace sq {

// LDS tile of one operand: rows of BKB bytes (2*BKB codes), stored as 16-byte chunks.
// Chunk c of row r sits at chunk slot r*CPR + (c ^ swz(r)).  The LDS of this part serves a
// 16-byte read of sixteen lanes per cycle from 64 banks (256 bytes): with swz(r) = (r / 2) % 8 for
// rows of 128 bytes (two rows per 256 bytes) and (r / 4) % 4 for rows of 64 bytes, the sixteen
// consecutive rows that read the same logical chunk land in sixteen different 16-byte bank groups
// (SQ_LDS_BANK_CONFLICT reads 0 for the kernel; with swz(r) = r % 8, which would be right for 32
// banks, it read 46 % of the LDS-active cycles -- at no difference in time: LDS is a third busy).
template <int BKB>
__device__ __forceinline__ int lds_chunk_slot(int row, int chunk)
{
    constexpr int CPR = BKB / 16;
    static_assert(CPR == 4 || CPR == 8, "tile row must be 64 or 128 bytes");
    const int swz = (CPR == 8) ? ((row >> 1) & 7) : ((row >> 2) & 3);
    return row * CPR + (chunk ^ swz);
}

// s_barrier without the memory fence of __syncthreads (which would wait for every outstanding
// global load).  The wave's own LDS accesses are drained first.
__device__ __forceinline__ void block_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Ring of NS stages, L loads per wave and tile, `rem` tiles exist beyond the one that must have
// landed (rem may be negative).  Loads complete in order, so that tile is in LDS once at most
// min(rem, NS - 2) * L loads are outstanding: wait for the largest count first and step down only
// in the last turns.  Then the LDS reads are drained and the waves meet at the barrier.
template <int L, int NS>
__device__ __forceinline__ void wait_tile_and_barrier(int rem)
{
    constexpr int D = NS - 2;
    static_assert(D >= 1 && D <= 4 && D * L < 64, "vmcnt is a 6-bit counter; at most four levels");
    constexpr int d0 = D, d1 = D > 1 ? D - 1 : 0, d2 = D > 2 ? D - 2 : 0, d3 = D > 3 ? D - 3 : 0;
    asm volatile("s_waitcnt vmcnt(%1)\n\t"
                 "s_cmp_ge_i32 %0, %2\n\t"
                 "s_cbranch_scc1 .Lsq_landed_%=\n\t"
                 "s_waitcnt vmcnt(%3)\n\t"
                 "s_cmp_ge_i32 %0, %4\n\t"
                 "s_cbranch_scc1 .Lsq_landed_%=\n\t"
                 "s_waitcnt vmcnt(%5)\n\t"
                 "s_cmp_ge_i32 %0, %6\n\t"
                 "s_cbranch_scc1 .Lsq_landed_%=\n\t"
                 "s_waitcnt vmcnt(%7)\n\t"
                 "s_cmp_ge_i32 %0, %8\n\t"
                 "s_cbranch_scc1 .Lsq_landed_%=\n\t"
                 "s_waitcnt vmcnt(0)\n"
                 ".Lsq_landed_%=:\n\t"
                 "s_waitcnt lgkmcnt(0)\n\t"
                 "s_barrier"
                 :
                 : "s"(rem), "n"(d0 * L), "n"(d0), "n"(d1 * L), "n"(d1), "n"(d2 * L), "n"(d2), "n"(d3 * L), "n"(d3)
                 : "memory", "scc");
}

// XCD-contiguous ids, then groups of 8 row-tiles walked column by column: the tiles resident on
// one XCD at a time share a few row panels and a few column panels in its L2.
__device__ __forceinline__ void tile_of_index(int index, int tiles_m, int tiles_n, int &bm, int &bn)
{
    const int id = xcd_contiguous_id(index, tiles_m * tiles_n);
    constexpr int GM = 8;
    const int group = id / (GM * tiles_n);
    const int gm = min(GM, tiles_m - group * GM);
    const int in_group = id - group * GM * tiles_n;
    bm = group * GM + in_group % gm;
    bn = in_group / gm;
}

__device__ __forceinline__ void tile_of_workgroup(int tiles_m, int tiles_n, int &bm, int &bn)
{
    tile_of_index((int)blockIdx.x, tiles_m, tiles_n, bm, bn);
}

}  // namespace sq
