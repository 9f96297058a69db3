// Insertion into the block hash table, shared by the builds that fill it: the
// slot of a key, and the node masks of the blocks an owner block's stencils
// touch.
#pragma once

#include "internal.h"

namespace mpmx {

// Claims or finds the slot of key K (Eqs. 23-25): a probed slot is read
// first and compare-and-swapped from EMPTY only when it is empty (most inserts
// find their block already claimed by another wave: each block is the owner
// or an upper neighbour of up to 2^d inserting waves).
// The claiming thread adds the slot to its tile's count.
__device__ __forceinline__ int hash_insert(const DevParams& P, uint64_t K) {
    unsigned s = (unsigned)mix64(K) & P.h_mask_bits;
    for (int r = 0; r < P.n_probe; ++r) {
        const uint64_t cur = __hip_atomic_load(&P.h_keys[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == K) return (int)s;
        if (cur == EMPTY_KEY) {
            const uint64_t old = atomicCAS((unsigned long long*)&P.h_keys[s], (unsigned long long)EMPTY_KEY,
                                           (unsigned long long)K);
            if (old == EMPTY_KEY) atomicAdd(&P.t_cnt[s / SCAN_TILE * LINE], 1u);
            if (old == EMPTY_KEY || old == K) return (int)s;
        }
        s = (s + 1) & P.h_mask_bits;
    }
    raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
    return -1;
}

// Node masks from the occupied base cells of a block.  With bit i + 4 j + 16 k
// for cell / node (i, j, k), the stencil of a base cell covers nodes +0..+2 on
// each axis; along one axis that is a dilation inside the block ("own") and a
// spill of cells 2 and 3 into nodes 0 and 1 of the upper neighbour ("spill").
// The node mask of neighbour d = (dx, dy, dz) is the composition of the per-axis
// own/spill maps selected by the bits of d.
__device__ __forceinline__ uint64_t own_x(uint64_t o) {
    return o | ((o << 1) & 0xEEEEEEEEEEEEEEEEull) | ((o << 2) & 0xCCCCCCCCCCCCCCCCull);
}
__device__ __forceinline__ uint64_t spill_x(uint64_t o) {
    return ((o >> 2) & 0x1111111111111111ull) | ((o >> 3) & 0x1111111111111111ull) |
           ((o >> 2) & 0x2222222222222222ull);
}
template <int DIM>
__device__ __forceinline__ uint64_t own_y(uint64_t o) {
    if (DIM == 2) return (o | (o << 4) | (o << 8)) & 0xFFFFull;
    return o | ((o << 4) & ~0x000F000F000F000Full) | ((o << 8) & ~0x00FF00FF00FF00FFull);
}
template <int DIM>
__device__ __forceinline__ uint64_t spill_y(uint64_t o) {
    if (DIM == 2) return ((o >> 8) & 0xFull) | ((o >> 12) & 0xFull) | ((o >> 8) & 0xF0ull);
    return ((o >> 8) & 0x000F000F000F000Full) | ((o >> 12) & 0x000F000F000F000Full) |
           ((o >> 8) & 0x00F000F000F000F0ull);
}
__device__ __forceinline__ uint64_t own_z(uint64_t o) { return o | (o << 16) | (o << 32); }
__device__ __forceinline__ uint64_t spill_z(uint64_t o) {
    return ((o >> 32) & 0xFFFFull) | ((o >> 48) & 0xFFFFull) | ((o >> 32) & 0xFFFF0000ull);
}

template <int DIM>
__device__ __forceinline__ uint64_t neighbour_mask(uint64_t occ, int d) {
    uint64_t o = (d & 1) ? spill_x(occ) : own_x(occ);
    if (DIM == 2) o &= 0xFFFFull;
    o = (d & 2) ? spill_y<DIM>(o) : own_y<DIM>(o);
    if (DIM == 3) o = (d & 4) ? spill_z(o) : own_z(o);
    return o;
}

// Empties the block hash: thread t of nt (Algorithm 5, initialisation).  LINKS:
// also the neighbours' slots, for insertions that store only the reached ones.
template <int NB, bool LINKS>
__device__ __forceinline__ void clear_hash(const DevParams& P, unsigned H, unsigned t, unsigned nt) {
    const unsigned tiles = (H + SCAN_TILE - 1) / SCAN_TILE;
    for (unsigned s = t; s < H; s += nt) {
        P.h_keys[s] = EMPTY_KEY;
        P.h_mask[s] = 0ull;
        P.h_start[s] = -1;
        P.h_end[s] = -1;
        if (P.h_entry) P.h_entry[s] = -1;
        if (LINKS)
#pragma unroll
            for (int d = 0; d < NB; d += 4) *(int4*)&P.h_nslot[(size_t)s * NB + d] = make_int4(-1, -1, -1, -1);
        if (s < tiles) P.t_cnt[s * LINE] = P.t_cnt[s * LINE + 1] = 0u;
    }
}

// Inserts block d of the 2^d blocks that the stencils of owner block `seg`
// (instance and linear block) with base cells `occ` can reach.  Returns its
// slot, -1 where it is not reached (or, with the overflow flag, where no slot
// was found).  d = 0 is the owner block itself.
template <int DIM>
__device__ __forceinline__ int insert_block(const DevParams& P, uint32_t seg, uint64_t occ, int d) {
    const uint64_t mymask = neighbour_mask<DIM>(occ, d);
    if (mymask == 0ull) return -1;
    int bc[3];
    linear_to_block<DIM>(P, seg & ((1u << P.blk_bits) - 1u), bc);
    const uint64_t K = block_key<DIM>(P, bc[0] + (d & 1), bc[1] + ((d >> 1) & 1), bc[2] + ((d >> 2) & 1),
                                      (int)(seg >> P.blk_bits));
    const int slot = hash_insert(P, K);
    if (slot >= 0) atomicOr((unsigned long long*)&P.h_mask[slot], (unsigned long long)mymask);
    return slot;
}

}  // namespace mpmx
