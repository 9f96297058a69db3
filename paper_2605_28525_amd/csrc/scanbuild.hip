// Scan-based active set (the paper's first construction, Methods 3.2 and
// Algorithms 1-4, here on the GPU): the alternative to the hash table of
// Algorithms 5-6.  It yields the same active blocks and node masks, with the
// compact index Phi in ascending block-key order.
//
//   k_sb_bbox   bounding box of the owner blocks of all particles: each of a
//               fixed number of workgroups reduces its share (wave shuffles,
//               then LDS) and writes one partial box, no atomics;
//   k_sb_box    one workgroup reduces the partial boxes; the mask domain is the
//               box grown by one block on each upper side (a stencil spills
//               only upward), its extents and volume m, all on the device (no
//               host read-back);
//   k_sb_zero   occupancy of the m blocks of the domain <- 0;
//   k_sb_occ    per owner block, the 64-bit occupancy of its base cells (lanes
//               of a wave with the same owner merged by ballot, one atomicOr);
//               from sorted keys it also records each owner segment's first and
//               one-past-last sorted position;
//   k_sb_flag   per block of the domain: active iff the OR over itself and its
//               2^d - 1 lower neighbours of the dilated occupancy (own part for
//               itself, spill part for the neighbours) is non-zero, a gather
//               with no atomics;
//   scan        exclusive scan of the flags -> compact index (Eq. 18);
//   k_sb_write  keys (Eq. 22) and node masks of the flagged blocks, in the
//               domain's order: i slowest, k fastest, which is ascending key
//               order (Eq. 22 packs i highest);
//   step build  (k_sb_write_blocks, k_sb_block_setup) the same into the
//               context's block tables, owner segments, upper and lower
//               neighbours looked up in the domain instead of the hash table;
//               after a counting sort (domains of up to TAB_MAX_IDS blocks) by
//               the shorter k_sbt_flag, k_sbt_write, k_sbt_link.
//
// The scratch (accumulators, occupancy, flags, Phi, segment bounds, scan
// partials) is passed in as an SbScratch: the context's own, allocated at
// create for the whole potential domain, or a fixed static device array.
#include <algorithm>
#include <climits>

#include "hash.h"
#include "../../include/mpm.h"

namespace mpmx {

// Owner block coordinates and base cell of particle i, from a sorted key or,
// with x != nullptr, from its position (the binning arithmetic of k_bin: base
// node floor(x/dx - 1/2) in float64, clamped into the grid).
template <int DIM>
__device__ __forceinline__ void sb_owner(const DevParams& P, const float* __restrict__ x,
                                         const uint32_t* __restrict__ keys, int n, int i, int* bc, int* cell) {
    if (x) {
        int b[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            double f = floor(index_arg(x[(size_t)a * n + i], P.inv_dx));
            if (!(f == f)) f = 0.0;
            f = fmin(fmax(f, 0.0), (double)(P.cells[a] - 2));
            b[a] = (int)f;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) bc[a] = b[a] >> 2;
        *cell = DIM == 3 ? ((b[0] & 3) | ((b[1] & 3) << 2) | ((b[2] & 3) << 4)) : ((b[0] & 3) | ((b[1] & 3) << 2));
        return;
    }
    const uint32_t k = keys[i];
    linear_to_block<DIM>(P, (k >> (2 * DIM)) & ((1u << P.blk_bits) - 1u), bc);
    *cell = (int)(k & ((1u << (2 * DIM)) - 1u));
}

// Domain index of block coordinates c (box-relative), i slowest, k fastest.
__device__ __forceinline__ long long sb_index(const SbBox& B, int c0, int c1, int c2) {
    return ((long long)c0 * B.ext[1] + c1) * B.ext[2] + c2;
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_bbox(DevParams P, const float* __restrict__ x,
                                                const uint32_t* __restrict__ keys, int n, int* __restrict__ bbp) {
    __shared__ int red[WG / 64][6];
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {-1, -1, -1};
    for (int i = blockIdx.x * WG + threadIdx.x; i < n; i += gridDim.x * WG) {
        int bc[3], cell;
        sb_owner<DIM>(P, x, keys, n, i, bc, &cell);
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            lo[a] = min(lo[a], bc[a]);
            hi[a] = max(hi[a], bc[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int m = 32; m >= 1; m >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], m));
            hi[a] = max(hi[a], __shfl_xor(hi[a], m));
        }
    }
    const int w = threadIdx.x >> 6;
    if (__lane_id() == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            red[w][a] = lo[a];
            red[w][3 + a] = hi[a];
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int t = threadIdx.x;
        int v = red[0][t];
        for (int q = 1; q < WG / 64; ++q) v = t < 3 ? min(v, red[q][t]) : max(v, red[q][t]);
        bbp[blockIdx.x * 8 + t] = v;
    }
}

// The bounding box from the partial boxes, and the extents of the mask domain;
// volume 0 when there is no particle or when it exceeds max_m (then too_big is
// set and nothing further is done).  The active-block total is set by the
// scan that follows.
template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_box(DevParams P, const int* __restrict__ bbp, int parts, SbBox* box,
                                               long long max_m) {
    __shared__ int red[WG / 64][6];
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {-1, -1, -1};
    for (int q = threadIdx.x; q < parts; q += WG) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = min(lo[a], bbp[q * 8 + a]);
            hi[a] = max(hi[a], bbp[q * 8 + 3 + a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int m = 32; m >= 1; m >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], m));
            hi[a] = max(hi[a], __shfl_xor(hi[a], m));
        }
    }
    const int w = threadIdx.x >> 6;
    if (__lane_id() == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            red[w][a] = lo[a];
            red[w][3 + a] = hi[a];
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int a = 0; a < 3; ++a) {
        box->lo[a] = red[0][a];
        box->hi[a] = red[0][3 + a];
        for (int q = 1; q < WG / 64; ++q) {
            box->lo[a] = min(box->lo[a], red[q][a]);
            box->hi[a] = max(box->hi[a], red[q][3 + a]);
        }
    }
    box->too_big = 0;
    long long m = 1;
    for (int a = 0; a < 3; ++a) {
        if (a >= DIM) {
            box->lo[a] = 0;
            box->ext[a] = 1;
            continue;
        }
        if (box->hi[a] < 0) {  // no particle
            m = 0;
            box->lo[a] = 0;
            box->ext[a] = 0;
            continue;
        }
        // owners lo..hi plus the upper neighbour, inside the potential domain
        box->ext[a] = min(box->hi[a] + 1, P.nblk[a] - 1) - box->lo[a] + 1;
        m *= box->ext[a];
    }
    if (m > max_m) {
        box->too_big = 1;
        m = 0;
    }
    box->m = (int)m;
}

__global__ __launch_bounds__(WG) void k_sb_zero(const SbBox* __restrict__ box, uint64_t* __restrict__ occ) {
    const int m = box->m;
    for (int t = blockIdx.x * WG + threadIdx.x; t < m; t += gridDim.x * WG) occ[t] = 0ull;
}

// Occupancy of each owner block's base cells; from sorted keys (x == nullptr)
// also the first and one-past-last sorted position of each owner segment.
template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_occ(DevParams P, const float* __restrict__ x,
                                               const uint32_t* __restrict__ keys, int n,
                                               const SbBox* __restrict__ box, uint64_t* __restrict__ occ,
                                               int* __restrict__ seg_lo, int* __restrict__ seg_hi) {
    const SbBox B = *box;
    if (B.m == 0) return;
    const int lane = __lane_id();
    for (int i0 = blockIdx.x * WG + (threadIdx.x & ~63); i0 < n; i0 += gridDim.x * WG) {
        const int i = i0 + lane;
        const bool valid = i < n;
        long long idx = -1;
        uint64_t bit = 0ull;
        if (valid) {
            int bc[3], cell;
            sb_owner<DIM>(P, x, keys, n, i, bc, &cell);
            idx = sb_index(B, bc[0] - B.lo[0], bc[1] - B.lo[1], bc[2] - B.lo[2]);
            bit = 1ull << cell;
            if (!x) {  // owner segment bounds of the sorted order
                const uint32_t seg = keys[i] >> (2 * DIM);
                if (i == 0 || (keys[i - 1] >> (2 * DIM)) != seg) seg_lo[idx] = i;
                if (i == n - 1 || (keys[i + 1] >> (2 * DIM)) != seg) seg_hi[idx] = i + 1;
            }
        }
        unsigned long long pending = __ballot(valid);
        while (pending) {  // one round per distinct owner block in the wave
            const int leader = __ffsll((long long)pending) - 1;
            const long long own = __shfl(idx, leader);
            const bool mine = valid && idx == own;
            const uint64_t mk = wave_or64(mine ? bit : 0ull);
            if (lane == leader) atomicOr((unsigned long long*)&occ[own], (unsigned long long)mk);
            pending &= ~__ballot(mine);
        }
    }
}

// Node mask of domain block (c0, c1, c2): its own dilated occupancy and the
// spills of its lower neighbours.
template <int DIM>
__device__ __forceinline__ uint64_t sb_mask_at(const SbBox& B, const uint64_t* __restrict__ occ, int c0, int c1,
                                               int c2) {
    constexpr int NB = 1 << DIM;
    uint64_t acc = 0ull;
#pragma unroll
    for (int d = 0; d < NB; ++d) {
        const int a0 = c0 - (d & 1), a1 = c1 - ((d >> 1) & 1), a2 = c2 - ((d >> 2) & 1);
        if (a0 < 0 || a1 < 0 || a2 < 0) continue;
        const uint64_t o = occ[sb_index(B, a0, a1, a2)];
        if (o) acc |= neighbour_mask<DIM>(o, d);
    }
    return acc;
}

__device__ __forceinline__ void sb_coords(const SbBox& B, int t, int* c) {
    c[2] = t % B.ext[2];
    const int r = t / B.ext[2];
    c[1] = r % B.ext[1];
    c[0] = r / B.ext[1];
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_flag(const SbBox* __restrict__ box, const uint64_t* __restrict__ occ,
                                                unsigned* __restrict__ flag) {
    const SbBox B = *box;
    for (int t = blockIdx.x * WG + threadIdx.x; t < B.m; t += gridDim.x * WG) {
        int c[3];
        sb_coords(B, t, c);
        flag[t] = sb_mask_at<DIM>(B, occ, c[0], c[1], c[2]) != 0ull ? 1u : 0u;
    }
}

// Keys and masks of the flagged blocks into caller arrays (the first cap).
template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_write(DevParams P, const SbBox* __restrict__ box,
                                                 const uint64_t* __restrict__ occ, const unsigned* __restrict__ flag,
                                                 const unsigned* __restrict__ phi, uint64_t* __restrict__ keys_out,
                                                 uint64_t* __restrict__ masks_out, int cap) {
    const SbBox B = *box;
    for (int t = blockIdx.x * WG + threadIdx.x; t < B.m; t += gridDim.x * WG) {
        if (!flag[t]) continue;
        const unsigned p = phi[t];
        if (p >= (unsigned)cap) continue;
        int c[3];
        sb_coords(B, t, c);
        keys_out[p] = block_key<DIM>(P, B.lo[0] + c[0], B.lo[1] + c[1], B.lo[2] + c[2], 0);
        masks_out[p] = sb_mask_at<DIM>(B, occ, c[0], c[1], c[2]);
    }
}

// Step build: the flagged blocks into the context's block tables in Phi order,
// with their owner segments; the block count and the capacity check.
template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_write_blocks(DevParams P, const SbBox* __restrict__ box,
                                                        const uint64_t* __restrict__ occ,
                                                        const unsigned* __restrict__ flag,
                                                        const unsigned* __restrict__ phi,
                                                        const int* __restrict__ seg_lo,
                                                        const int* __restrict__ seg_hi) {
    const SbBox B = *box;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        P.ctr->n_touched = (int)B.total;
        P.ctr->nb = min((int)B.total, P.block_cap);
        P.ctr->n_work = 0;
        if ((int)B.total > P.block_cap) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
    }
    for (int t = blockIdx.x * WG + threadIdx.x; t < B.m; t += gridDim.x * WG) {
        if (!flag[t]) continue;
        const unsigned p = phi[t];
        if (p >= (unsigned)P.block_cap) continue;
        int c[3];
        sb_coords(B, t, c);
        P.b_keys[p] = block_key<DIM>(P, B.lo[0] + c[0], B.lo[1] + c[1], B.lo[2] + c[2], 0);
        P.b_mask[p] = sb_mask_at<DIM>(B, occ, c[0], c[1], c[2]);
        const bool owns = occ[t] != 0ull;
        const int st = owns ? seg_lo[t] : -1;
        P.b_start[p] = st;
        P.b_count[p] = owns ? seg_hi[t] - st : 0;
    }
}

// Compact index of the domain block at box-relative c, -1 outside the domain
// or inactive (or past the capacity).
__device__ __forceinline__ int sb_phi_at(const DevParams& P, const SbBox& B, const unsigned* __restrict__ flag,
                                         const unsigned* __restrict__ phi, int c0, int c1, int c2) {
    if (c0 < 0 || c1 < 0 || c2 < 0 || c0 >= B.ext[0] || c1 >= B.ext[1] || c2 >= B.ext[2]) return -1;
    const long long t = sb_index(B, c0, c1, c2);
    if (!flag[t]) return -1;
    const unsigned p = phi[t];
    return p < (unsigned)P.block_cap ? (int)p : -1;
}

// Upper and lower neighbours (looked up in the domain) and
// the chunk count of each block.
template <int DIM>
__global__ __launch_bounds__(WG) void k_sb_block_setup(DevParams P, const SbBox* __restrict__ box,
                                                       const unsigned* __restrict__ flag,
                                                       const unsigned* __restrict__ phi) {
    constexpr int NB = 1 << DIM;
    const SbBox B = *box;
    const int nb = P.ctr->nb;
    for (int b = blockIdx.x * WG + threadIdx.x; b < nb; b += gridDim.x * WG) {
        int bc[3], inst;
        unblock_key<DIM>(P, P.b_keys[b], bc, &inst);
        const int c0 = bc[0] - B.lo[0], c1 = bc[1] - B.lo[1], c2 = bc[2] - B.lo[2];
        P.b_nbr[b * NB] = b;
#pragma unroll
        for (int d = 1; d < NB; ++d)
            P.b_nbr[b * NB + d] = sb_phi_at(P, B, flag, phi, c0 + (d & 1), c1 + ((d >> 1) & 1), c2 + ((d >> 2) & 1));
        if (P.b_lo) {
            P.b_lo[b * NB] = P.b_count[b] > 0 ? b : -1;
#pragma unroll
            for (int d = 1; d < NB; ++d) {
                const int lo = sb_phi_at(P, B, flag, phi, c0 - (d & 1), c1 - ((d >> 1) & 1), c2 - ((d >> 2) & 1));
                P.b_lo[b * NB + d] = (lo >= 0 && P.b_count[lo] > 0) ? lo : -1;
            }
        }
        P.b_chunks[b] = (unsigned)((P.b_count[b] + P.chunk - 1) / P.chunk);
    }
}

namespace {
int sb_grid(long long items, int cap_wgs) {
    long long g = (items + WG - 1) / WG;
    if (g < 1) g = 1;
    if (g > cap_wgs) g = cap_wgs;
    return (int)g;
}

// Bounding box, domain, occupancy, flags and their scan: the part shared by
// the query and the step build.  x != nullptr: bins the positions on the fly;
// else reads sorted keys.
hipError_t sb_mark(const DevParams& P, const float* x, const uint32_t* keys, int n, const SbScratch& S,
                   hipStream_t s) {
    const int gp = sb_grid(n, 4096);
    const int gm = sb_grid(S.max_m, 8192);
    if (P.dim == 3) {
        k_sb_bbox<3><<<SB_BBOX_WGS, WG, 0, s>>>(P, x, keys, n, S.bbp);
        k_sb_box<3><<<1, WG, 0, s>>>(P, S.bbp, SB_BBOX_WGS, S.box, S.max_m);
        k_sb_zero<<<gm, WG, 0, s>>>(S.box, S.occ);
        if (n > 0) k_sb_occ<3><<<gp, WG, 0, s>>>(P, x, keys, n, S.box, S.occ, S.seg_lo, S.seg_hi);
        k_sb_flag<3><<<gm, WG, 0, s>>>(S.box, S.occ, S.flag);
    } else {
        k_sb_bbox<2><<<SB_BBOX_WGS, WG, 0, s>>>(P, x, keys, n, S.bbp);
        k_sb_box<2><<<1, WG, 0, s>>>(P, S.bbp, SB_BBOX_WGS, S.box, S.max_m);
        k_sb_zero<<<gm, WG, 0, s>>>(S.box, S.occ);
        if (n > 0) k_sb_occ<2><<<gp, WG, 0, s>>>(P, x, keys, n, S.box, S.occ, S.seg_lo, S.seg_hi);
        k_sb_flag<2><<<gm, WG, 0, s>>>(S.box, S.occ, S.flag);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return scan_exclusive(S.flag, S.phi, (int)S.max_m, &S.box->m, S.partials, &S.box->total, s);
}
}  // namespace

size_t sb_scratch_bytes(long long max_m) {
    // segment bounds (2 x i32 per block) are allocated by the step build's owner
    return sb_scratch_size(max_m);
}

SbScratch sb_carve(void* base, long long max_m, int* seg_lo, int* seg_hi) {
    SbScratch S{};
    char* p = (char*)base;
    S.box = (SbBox*)p;
    p += 256;
    S.bbp = (int*)p;
    p += (size_t)SB_BBOX_WGS * 8 * sizeof(int);
    S.occ = (uint64_t*)p;
    p += (size_t)max_m * 8;
    S.flag = (unsigned*)p;
    p += (size_t)max_m * 4;
    S.phi = (unsigned*)p;
    p += (size_t)max_m * 4;
    S.partials = (unsigned*)p;
    S.max_m = max_m;
    S.seg_lo = seg_lo;
    S.seg_hi = seg_hi;
    return S;
}

hipError_t launch_scan_active(const DevParams& P, const float* x, int n, const SbScratch& S, uint64_t* keys_out,
                              uint64_t* masks_out, int cap, hipStream_t s) {
    hipError_t e = sb_mark(P, x, nullptr, n, S, s);
    if (e != hipSuccess || cap <= 0) return e;
    const int gm = sb_grid(S.max_m, 8192);
    if (P.dim == 3)
        k_sb_write<3><<<gm, WG, 0, s>>>(P, S.box, S.occ, S.flag, S.phi, keys_out, masks_out, cap);
    else
        k_sb_write<2><<<gm, WG, 0, s>>>(P, S.box, S.occ, S.flag, S.phi, keys_out, masks_out, cap);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The step build after a counting sort (tabsort.hip), which leaves per owner
// block its occupied cells, particles, first position and entry, and per tile of
// its table a bounding box: nothing is read per particle, no mask is gathered
// twice, and the compaction writes the block tables and the work items, as the
// hash build's does.  Three launches, each a chain of two or three accesses:
// 8.0, 5.5 and 3.8 us of a step of 312,500 particles; from the sorted keys it
// took twelve, 54 us.
//
//   k_sbt_flag   box from the tiles' boxes; node masks of the domain's blocks
//                (a gather over each block's lower neighbours); per tile of
//                the domain the active blocks and their work items;
//   k_sbt_write  Phi, the block tables in its order, the work items;
//   k_sbt_link   neighbour tables; empties the sort's table.

// Linear block index (the sort's) of the domain's block at box-relative c.
template <int DIM>
__device__ __forceinline__ int sb_linear(const DevParams& P, const SbBox& B, int c0, int c1, int c2) {
    const int x = B.lo[0] + c0, y = B.lo[1] + c1, z = B.lo[2] + c2;
    return DIM == 3 ? (z * P.nblk[1] + y) * P.nblk[0] + x : y * P.nblk[0] + x;
}

// Blocks of the domain per tile: small, so that the few tiles of an ordinary
// box still spread over the chip (their loads are dependent chains).
constexpr int SBT_ITEMS = 2, SBT_TILE = WG * SBT_ITEMS;

template <int DIM>
__global__ __launch_bounds__(WG) void k_sbt_flag(DevParams P, TabSort T, SbScratch S) {
    constexpr int NB = 1 << DIM;
    __shared__ int red[WG / 64][6];
    __shared__ unsigned lds[WG / 64];
    SbBox B;
    {
        int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {-1, -1, -1};
        const int tiles = (T.ids + SCAN_TILE - 1) / SCAN_TILE;
        for (int q = threadIdx.x; q < tiles; q += WG) {
            const int4 l = *(const int4*)&T.box[8 * q], h = *(const int4*)&T.box[8 * q + 4];
            lo[0] = min(lo[0], l.x);
            lo[1] = min(lo[1], l.y);
            lo[2] = min(lo[2], l.z);
            hi[0] = max(hi[0], h.x);
            hi[1] = max(hi[1], h.y);
            hi[2] = max(hi[2], h.z);
        }
        box_reduce(lo, hi, red);
        long long m = 1;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            // owners lo..hi plus the upper neighbour, inside the potential domain
            const bool none = hi[a] < 0;
            B.lo[a] = a < DIM && !none ? lo[a] : 0;
            B.hi[a] = hi[a];
            B.ext[a] = a >= DIM ? 1 : none ? 0 : min(hi[a] + 1, P.nblk[a] - 1) - lo[a] + 1;
            m *= B.ext[a];
        }
        B.m = (int)m;
        B.too_big = 0;
        B.total = 0u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *S.box = B;
    for (int tile = blockIdx.x; tile * SBT_TILE < B.m; tile += gridDim.x) {
        // (every load at a clamped index and masked afterwards: behind the bounds'
        // branches they went out one by one, 8.6 us; an empty block's masks, most of
        // the box, are still skipped)
        uint64_t o[SBT_ITEMS][NB];
        unsigned own[SBT_ITEMS], in[SBT_ITEMS];
#pragma unroll
        for (int j = 0; j < SBT_ITEMS; ++j) {
            int c[3];
            sb_coords(B, min(tile * SBT_TILE + j * WG + (int)threadIdx.x, (int)B.m - 1), c);
            in[j] = 0u;
#pragma unroll
            for (int d = 0; d < NB; ++d) {
                const int a0 = c[0] - (d & 1), a1 = c[1] - ((d >> 1) & 1), a2 = c[2] - ((d >> 2) & 1);
                const int id = sb_linear<DIM>(P, B, max(a0, 0), max(a1, 0), max(a2, 0));
                o[j][d] = T.occ[id];
                if (d == 0) own[j] = T.cnt[id];
                in[j] |= (a0 | a1 | a2) >= 0 ? 1u << d : 0u;
            }
        }
        unsigned act = 0u, items = 0u;
#pragma unroll
        for (int j = 0; j < SBT_ITEMS; ++j) {
            const int t = tile * SBT_TILE + j * WG + (int)threadIdx.x;
            uint64_t mask = 0ull;
#pragma unroll
            for (int d = 0; d < NB; ++d)
                if ((in[j] >> d & 1u) && o[j][d]) mask |= neighbour_mask<DIM>(o[j][d], d);
            if (t >= B.m) continue;
            S.occ[t] = mask;
            act += mask != 0ull ? 1u : 0u;
            items += block_chunks(P, (int)own[j]);
        }
        unsigned ta, ti;
        wg_excl_scan(act, lds, &ta);
        wg_excl_scan(items, lds, &ti);
        if (threadIdx.x == 0) {
            T.part[2 * tile] = ta;  // (the sort has finished with its tile sums)
            T.part[2 * tile + 1] = ti;
        }
    }
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_sbt_write(DevParams P, TabSort T, SbScratch S) {
    constexpr int NW = WG / 64;
    __shared__ unsigned short list[SBT_TILE];  // active blocks of the tile, ascending
    __shared__ unsigned red[NW][4], wcnt[NW * SBT_ITEMS], lds[NW];
    const SbBox B = *S.box;
    const int lane = __lane_id(), wv = threadIdx.x >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int tiles = (B.m + SBT_TILE - 1) / SBT_TILE;
    bool over = false;
    // (tile 0 is always visited: its workgroup sets the counters)
    for (int tile = blockIdx.x; tile == 0 || tile < tiles; tile += gridDim.x) {
        uint64_t k[SBT_ITEMS];
#pragma unroll
        for (int j = 0; j < SBT_ITEMS; ++j) {
            const int t = tile * SBT_TILE + j * WG + (int)threadIdx.x;
            k[j] = t < B.m ? S.occ[t] : 0ull;
        }
        unsigned sum[4] = {0u, 0u, 0u, 0u};
        for (int i = threadIdx.x; i < tiles; i += WG) {
            const uint2 p = *(const uint2*)&T.part[2 * i];
            sum[0] += i < tile ? p.x : 0u;
            sum[1] += i < tile ? p.y : 0u;
            sum[2] += p.x;
            sum[3] += p.y;
        }
        unsigned long long occ[SBT_ITEMS];
#pragma unroll
        for (int j = 0; j < SBT_ITEMS; ++j) {
            occ[j] = __ballot(k[j] != 0ull);
            if (lane == 0) wcnt[j * NW + wv] = (unsigned)__popcll(occ[j]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] += __shfl_xor(sum[q], o);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) red[wv][q] = sum[q];
        __syncthreads();
        const unsigned mine = lane < NW * SBT_ITEMS ? wcnt[lane] : 0u;
        const unsigned inc = wave_incl_scan(mine);
        const int n_act = readlane32((int)inc, 63);
        unsigned phi0 = 0u, it0 = 0u, total = 0u, items = 0u;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            phi0 += red[q][0];
            it0 += red[q][1];
            total += red[q][2];
            items += red[q][3];
        }
#pragma unroll
        for (int j = 0; j < SBT_ITEMS; ++j) {
            const int q = j * NW + wv, t = tile * SBT_TILE + j * WG + (int)threadIdx.x;
            const unsigned r = (unsigned)__shfl((int)(inc - mine), q) + (unsigned)__popcll(occ[j] & lt);
            const bool on = k[j] != 0ull;
            if (on) list[r] = (unsigned short)(j * WG + threadIdx.x);
            if (t < B.m) S.phi[t] = on && phi0 + r < (unsigned)P.block_cap ? phi0 + r : ~0u;
        }
        __syncthreads();
#pragma unroll 1
        for (int r0 = 0; r0 < n_act; r0 += WG) {
            const int r = r0 + (int)threadIdx.x;
            const bool on = r < n_act;
            const int t = on ? tile * SBT_TILE + list[r] : 0;
            const unsigned p = phi0 + (unsigned)r;
            int c[3], cnt = 0, st = -1, ent = -1;
            uint64_t mask = 0ull;
            sb_coords(B, t, c);
            if (on) {
                const int id = sb_linear<DIM>(P, B, c[0], c[1], c[2]);
                mask = S.occ[t];
                cnt = (int)T.cnt[id];
                const int first = (int)T.start[id], e = T.eidx[id];  // of an earlier build where cnt is 0
                if (cnt > 0) {
                    st = first;
                    ent = e < P.row_cap ? e : -1;
                }
            }
            const unsigned chunks = block_chunks(P, cnt);
            unsigned tot;
            const unsigned w = it0 + wg_excl_scan(chunks, lds, &tot);
            it0 += tot;
            if (on && p < (unsigned)P.block_cap) {
                P.b_keys[p] = block_key<DIM>(P, B.lo[0] + c[0], B.lo[1] + c[1], B.lo[2] + c[2], 0);
                P.b_mask[p] = mask;
                P.b_start[p] = st;
                P.b_count[p] = cnt;
                P.b_chunks[p] = chunks;
                if (P.b_entry) P.b_entry[p] = ent;
                for (unsigned q = 0; q < chunks; ++q) {
                    if (w + q >= (unsigned)P.work_cap) {
                        over = true;
                        break;
                    }
                    P.w_block[w + q] = (int)p;
                    P.w_start[w + q] = st + (int)q * P.chunk;
                    P.w_end[w + q] = min(st + ((int)q + 1) * P.chunk, st + cnt);
                }
            } else if (on) {
                over = true;
            }
        }
        if (tile == 0 && threadIdx.x == 0) {
            S.box->total = total;
            P.ctr->n_touched = (int)total;
            P.ctr->nb = min((int)total, P.block_cap);
            // the items of blocks past the capacity were not written: no work then
            P.ctr->n_work = total <= (unsigned)P.block_cap ? (int)items : 0;
        }
        __syncthreads();
    }
    if (over) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
}

// 2^d lanes per block, one for each upper and the lower neighbour opposite.
template <int DIM>
__global__ __launch_bounds__(WG) void k_sbt_link(DevParams P, TabSort T, SbScratch S) {
    constexpr int NB = 1 << DIM;
    const SbBox B = *S.box;
    const int nb = P.ctr->nb, ne = min(*T.n_ent, T.ent_cap);
    const int t0 = blockIdx.x * WG + threadIdx.x, tn = gridDim.x * WG, d = t0 % NB;
    auto phi_at = [&](int c0, int c1, int c2) {
        if (c0 < 0 || c1 < 0 || c2 < 0 || c0 >= B.ext[0] || c1 >= B.ext[1] || c2 >= B.ext[2]) return -1;
        return (int)S.phi[sb_index(B, c0, c1, c2)];
    };
    const int d0 = d & 1, d1 = (d >> 1) & 1, d2 = (d >> 2) & 1;
    for (int b = t0 / NB; b < nb; b += tn / NB) {
        int bc[3], inst;
        unblock_key<DIM>(P, P.b_keys[b], bc, &inst);
        const int c0 = bc[0] - B.lo[0], c1 = bc[1] - B.lo[1], c2 = bc[2] - B.lo[2];
        const int up = phi_at(c0 + d0, c1 + d1, c2 + d2);
        const int lo = phi_at(c0 - d0, c1 - d1, c2 - d2);
        P.b_nbr[(size_t)b * NB + d] = up;
        P.b_lo[(size_t)b * NB + d] = lo >= 0 && P.b_count[lo] > 0 ? lo : -1;
    }
    for (int e = t0; e < ne; e += tn) {  // the table is left empty
        const unsigned id = T.ent[e].x;
        T.cnt[id] = 0u;
        T.occ[id] = 0ull;
    }
}

hipError_t launch_build_scan_tab(const DevParams& P, const TabSort& T, const SbScratch& S, hipStream_t s) {
    // one workgroup per tile of the largest domain, up to what the chip holds
    const int gt = (int)std::min<long long>((S.max_m + SBT_TILE - 1) / SBT_TILE, 2048);
    const int gl = (int)std::min<long long>((((long long)P.block_cap << P.dim) + WG - 1) / WG, 2048);
    if (P.dim == 3) {
        k_sbt_flag<3><<<gt, WG, 0, s>>>(P, T, S);
        k_sbt_write<3><<<gt, WG, 0, s>>>(P, T, S);
        k_sbt_link<3><<<gl, WG, 0, s>>>(P, T, S);
    } else {
        k_sbt_flag<2><<<gt, WG, 0, s>>>(P, T, S);
        k_sbt_write<2><<<gt, WG, 0, s>>>(P, T, S);
        k_sbt_link<2><<<gl, WG, 0, s>>>(P, T, S);
    }
    return hipGetLastError();
}

hipError_t launch_build_scan(const DevParams& P, const uint32_t* skeys, int n, const SbScratch& S,
                             unsigned* partials, hipStream_t s) {
    hipError_t e = sb_mark(P, nullptr, skeys, n, S, s);
    if (e != hipSuccess) return e;
    const int gm = sb_grid(S.max_m, 8192);
    const int gb = sb_grid(P.block_cap, 2048);
    if (P.dim == 3) {
        k_sb_write_blocks<3><<<gm, WG, 0, s>>>(P, S.box, S.occ, S.flag, S.phi, S.seg_lo, S.seg_hi);
        k_sb_block_setup<3><<<gb, WG, 0, s>>>(P, S.box, S.flag, S.phi);
    } else {
        k_sb_write_blocks<2><<<gm, WG, 0, s>>>(P, S.box, S.occ, S.flag, S.phi, S.seg_lo, S.seg_hi);
        k_sb_block_setup<2><<<gb, WG, 0, s>>>(P, S.box, S.flag, S.phi);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_work_items(P, partials, s);
}

}  // namespace mpmx
