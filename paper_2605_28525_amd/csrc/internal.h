// Internal declarations of the sparse-grid MPM library (gfx950, wave64).
//
// Device data layout (all in HBM, owned by the context):
//   sort      key/value ping-pong buffers, u32 x max_particles each; per-tile
//             digit histograms;
//   hash      H slots: packed block key (u64, EMPTY = ~0), node mask (u64),
//             compact index (i32), first/one-past-last sorted particle of the
//             block's owner segment (i32), the slots of the 2^d blocks its
//             stencils reach (i32 each);
//   blocks    block_capacity entries in compact order Phi: key, node mask,
//             2^d neighbour compact indices (upper neighbours), owner segment
//             start and length, P2G/G2P chunk count and offset;
//   work      (block, first, last) particle ranges of at most CHUNK particles;
//   grid      block_capacity * 4^d nodes, one float4 per node (p_x, p_y, p_z, m),
//             then (v_x, v_y, v_z, m) after the grid update.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mpm.h"

namespace mpmx {

constexpr int WG = 256;            // workgroup size of every kernel (4 wave64s)
constexpr int BLK = 4;             // block edge B (Methods 3.2)
constexpr int KEY_M = 21;          // bits per packed coordinate (Eq. 22)
constexpr int64_t KEY_BIAS = 1 << 20;
constexpr uint64_t EMPTY_KEY = ~0ull;

constexpr int SORT_ITEMS = 16;                 // keys per thread per radix tile
constexpr int SORT_TILE = WG * SORT_ITEMS;     // 4096 keys per tile
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = WG * SCAN_ITEMS;     // 2048 values per scan tile
constexpr int MIN_CHUNK = 64;                  // smallest particles-per-work-item setting
constexpr int MAX_CHUNK = 768;                 // largest (G2P stages a work item in LDS)
// Particles a G2P workgroup of gs threads stages per work item: three per
// thread at 256 threads (a full 4^3 block of 8-per-cell material, slightly
// compressed, stays one item), two per thread below.
constexpr int g2p_max_items(int gs) { return (gs == 256 ? 3 : 2) * gs; }

struct DevCounters {
    int nb;          // active blocks (compact count, <= capacity)
    int n_touched;   // occupied hash slots (may exceed capacity on overflow)
    int n_work;      // P2G/G2P work items
    unsigned flags;  // sticky MPM_FLAG_* bits
    int rs_n_new;    // incremental re-sort: blocks without a previous slot
    int rs_new_pos;  //   particles of the new blocks placed so far
    int pad[2];
};

constexpr int RS_TILE = 256;  // entries per partial sum of the re-sort's particle counts
// Words between counters that many workgroups add to: one cache line each.
// Adds to one line from several XCDs are served one after another, 15-20 ns
// each (12,500 adds to a single word took 200 us, a few thousand to counters
// sharing a line 40 us).
constexpr int LINE = 32;
// Particle count up to which the short passes of a build are folded into their
// neighbours (the re-sort's scan into the placement, the neighbour tables into
// P2G).  Below it a launch and a pass's latency are what they cost; above it
// the folded forms' extra loads cost more (2.5 M particles: placement 18.9 us
// against 14.0 + 9.5 for the scan, P2G +3 us against a 7 us pass; 20 M: 82
// against 68 + 9, P2G +30 us against 10).
constexpr int FOLD_MAX_N = 1 << 22;
// And blocks (what the host knows of their number is the capacity): the folded
// scan's loads grow with the square of the blocks, of which scattered particles
// have several each.  Steps of 65,536 / 131,072 / 262,144 particles scattered over
// 208,556 / 418,253 / 774,874 blocks in 1021 / 1961 / 4175 us folded, 970 / 1733 /
// 3273 not; 262,144 particles in 1000 blocks with room for 524,288 in 79 and 84.
constexpr int FOLD_MAX_BLOCKS = 1 << 18;
// Tiles of the hash table up to which each tile of the compaction adds up the
// counts of the tiles before it, a line each; above, one workgroup makes their
// running sums first.  Steps of 262,144 particles with a table of 2^21 / 2^22 / 2^23 /
// 2^24 / 2^25 slots (2048 in a tile) in 76 / 84 / 93 / 113 / 190 us, without the extra
// launch 73 / 90 / 136 / 321 / 1120.
constexpr int FOLD_MAX_TILES = 1024;

// Up to this many particles mpm_step leaves P2G's second pass to G2P, except in
// its last step, whose grid stays readable: a launch less, against nodes formed
// by each block that reads them.  Whole steps of 4,096 / 32,768 / 65,536 / 131,072 /
// 262,144 / 2,097,152 particles in 56 / 59 / 61 / 74 / 80 / 290 us, with the pass 57 /
// 61 / 62 / 73 / 79 / 267; in a graph of 25,600 53 against 56, of 4,096 in 2D
// 38 against 40 (all with 2^d particles per cell; of 64,000 with 1 / 27 per cell 71 / 78
// against 67 / 81, of 65,536 in 2D with 1 81 against 72).
constexpr int G2P_GATHER_MAX_N = 1 << 16;
// And where contexts have room for at most as many blocks: 65,536 particles
// scattered over 129,339 blocks (2D) in 464 us, with the pass 382; over 208,556 (3D)
// 972 and 909.
constexpr int G2P_GATHER_MAX_BLOCKS = 1 << 16;

// Per-instance material and step constants (one entry for a single simulation).
struct InstMat {
    float mu, lam, alpha, dp_coef;
    float dt, p_mass, p_vol0, E;
    float dalpha_dphi, pad[3];
};

constexpr int MAX_INSTANCES = 64;
constexpr int ENS_KEY_M = 19;                 // ensemble block keys: bits per coordinate
constexpr int64_t ENS_KEY_BIAS = 1 << 18;
constexpr int ENS_INST_SHIFT = 57;            // instance id in bits 57..62

struct DevParams {
    int dim;
    int cells[3];
    int nblk[3];          // blocks per axis over the node range [0, cells]
    int dense;
    double dx, inv_dx;
    float dxf, inv_dxf, dt;
    float g[3];
    float mu, lam, alpha, dp_coef;   // Lame, DP cone alpha, (d lambda + 2 mu)/(2 mu)
    int model;
    float p_mass, p_vol0;
    int bound;
    int bc[3][2];
    const float* heightmap;
    float mu_terrain;
    int has_terrain;
    // hash table
    uint64_t* h_keys;
    uint64_t* h_mask;
    int* h_vals;
    int* h_start;
    int* h_end;
    int* h_nslot;           // hash-built tables: per slot of an owner block, the slots of the 2^d
                            // blocks its stencils reach (d = 0: itself; -1: not reached)
    unsigned* t_cnt;        // per SCAN_TILE slots, LINE words apart: occupied ones, work items; in large
                            // tables also their sums over the tiles before (a line past the last: over all)
    unsigned h_mask_bits;   // H - 1
    int n_probe;
    // compact blocks
    uint64_t* b_keys;
    uint64_t* b_mask;
    int* b_nbr;
    int* b_start;
    int* b_count;
    unsigned* b_chunks;
    unsigned* b_chunk_off;
    int* b_hs;              // hash slot of each compact block (null: the build makes b_nbr, b_lo itself)
    int block_cap;
    // work items
    int* w_block;
    int* w_start;
    int* w_end;
    int work_cap;
    int chunk;
    // grid
    float4* grid;
    float4* tiles;        // sparse P2G: each block's (4+2)^d node tile, block-major
    int* b_lo;            // sparse P2G: 2^d lower neighbours (d = 0: the block) owning particles, else -1
    DevCounters* ctr;
    // reverse mode (allocated with MPM_FLAG_ADJOINT)
    float4* grid_u;      // pre-boundary nodal velocity u = p/m + dt g, and m
    float4* grid_bar;    // adjoint of the nodal velocity, then (p_bar, m_bar)
    float* adj_scratch;  // per G2P output position: v'_bar (d), B_bar (d*d), W_bar (d*d), x (d); plane stride n
    float* adj_part;     // per workgroup of the reverse G2P: dL/dE, dL/dalpha
    float* param_bar;    // accumulated dL/dE, dL/dphi (per degree)
    float E;
    float dalpha_dphi;   // d alpha / d phi, per degree
    // incremental re-sort (resort.hip): per entry (previous block, then new
    // block) and base cell, NC = 4^d columns
    uint32_t* rs_stay;    // stayers per previous block and cell
    uint32_t* rs_in;      // movers per entry and cell (counted down to zero as they are placed)
    uint32_t* rs_off;     // first sorted position per entry and cell
    unsigned* rs_cnt;     // particles per entry (stayers from G2P or the count pass, plus movers)
    unsigned* rs_start;   // first sorted position per entry
    int* rs_nslot;        // h_nslot's row of each entry
    uint64_t* rs_occ;     // base cells holding particles, per entry
    uint32_t* rs_oldblk;  // owner-block part of the sort key of each entry (~0: empty previous block)
    uint64_t* nh_keys;    // second hash table (same size as the block table): blocks
    uint32_t* nh_cnt;     //   with no previous slot, their movers per cell,
    int* nh_idx;          //   their entry index
    uint32_t* nh_owner;   //   and the owner-block part of their sort key
    uint32_t* rs_new;     // second-table slots in the order of their claims (block_cap entries)
    unsigned* rs_tile;    // particles per RS_TILE previous blocks (sums of rs_cnt), LINE words apart; null
                          // above FOLD_MAX_N particles or FOLD_MAX_BLOCKS blocks
    unsigned* it_mov;     // movers of each work item, listed from the item's first position on
    int* h_entry;         // the sort's entry of each hash slot's owner block (-1: none)
    int* b_entry;         // the sort's entry of each compact block (-1: none): its cell
                          // ranges are the entry's row of rs_off
    int row_cap;          // rows of rs_off and rs_nslot (0: none)
    const uint4* d_ent;   // dense grids, after a counting sort: the occupied blocks (TabSort::ent) and their
    const int* d_n;       // number; null after a radix sort
    // ensembles
    int n_inst;          // 1 = single simulation
    int blk_bits;        // bits of the linear block id inside the sort key
    const InstMat* inst; // device table, n_inst entries
};

// ---------------------------------------------------------------------------
// device helpers
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    // SplitMix64 output function (Steele, Lea, Flood 2014), a 64-bit mixer of
    // the kind cited for Eq. 23.
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

template <int DIM>
__device__ __forceinline__ uint64_t pack_key(int bx, int by, int bz) {
    // Eq. 22: ((i + b) << 2m) | ((j + b) << m) | (k + b); 2D packs (i, j) low.
    if (DIM == 3)
        return ((uint64_t)(bx + KEY_BIAS) << (2 * KEY_M)) | ((uint64_t)(by + KEY_BIAS) << KEY_M) |
               (uint64_t)(bz + KEY_BIAS);
    return ((uint64_t)(bx + KEY_BIAS) << KEY_M) | (uint64_t)(by + KEY_BIAS);
}

template <int DIM>
__device__ __forceinline__ void unpack_key(uint64_t k, int* b) {
    const uint64_t m = (1ull << KEY_M) - 1;
    if (DIM == 3) {
        b[0] = (int)((k >> (2 * KEY_M)) & m) - (int)KEY_BIAS;
        b[1] = (int)((k >> KEY_M) & m) - (int)KEY_BIAS;
        b[2] = (int)(k & m) - (int)KEY_BIAS;
    } else {
        b[0] = (int)((k >> KEY_M) & m) - (int)KEY_BIAS;
        b[1] = (int)(k & m) - (int)KEY_BIAS;
        b[2] = 0;
    }
}

// Block key with the instance folded in.  A single simulation uses Eq. 22
// as printed (m = 21, bias 2^20); an ensemble uses m = 19 (bias 2^18) and puts
// the instance id in bits 57-62, which keeps 3m + 6 <= 63.
template <int DIM>
__device__ __forceinline__ uint64_t block_key(const DevParams& P, int bx, int by, int bz, int inst) {
    if (P.n_inst <= 1) return pack_key<DIM>(bx, by, bz);
    const uint64_t ib = (uint64_t)inst << ENS_INST_SHIFT;
    if (DIM == 3)
        return ib | ((uint64_t)(bx + ENS_KEY_BIAS) << (2 * ENS_KEY_M)) | ((uint64_t)(by + ENS_KEY_BIAS) << ENS_KEY_M) |
               (uint64_t)(bz + ENS_KEY_BIAS);
    return ib | ((uint64_t)(bx + ENS_KEY_BIAS) << ENS_KEY_M) | (uint64_t)(by + ENS_KEY_BIAS);
}

template <int DIM>
__device__ __forceinline__ void unblock_key(const DevParams& P, uint64_t k, int* b, int* inst) {
    if (P.n_inst <= 1) {
        unpack_key<DIM>(k, b);
        *inst = 0;
        return;
    }
    const uint64_t m = (1ull << ENS_KEY_M) - 1;
    *inst = (int)((k >> ENS_INST_SHIFT) & 63u);
    if (DIM == 3) {
        b[0] = (int)((k >> (2 * ENS_KEY_M)) & m) - (int)ENS_KEY_BIAS;
        b[1] = (int)((k >> ENS_KEY_M) & m) - (int)ENS_KEY_BIAS;
        b[2] = (int)(k & m) - (int)ENS_KEY_BIAS;
    } else {
        b[0] = (int)((k >> ENS_KEY_M) & m) - (int)ENS_KEY_BIAS;
        b[1] = (int)(k & m) - (int)ENS_KEY_BIAS;
        b[2] = 0;
    }
}

// Base node floor(x * (1/dx) - 1/2) in float64, multiply and subtract rounded
// separately (no contraction), and the fractional offset s - floor(s).
__device__ __forceinline__ double index_arg(float x, double inv_dx) {
#pragma clang fp contract(off)
    double s = (double)x * inv_dx;
    return s - 0.5;
}

// Sort key of one particle (binning, a1): base node floor(x/dx - 1/2) per axis
// in float64, clamped into the grid with MPM_FLAG_DOMAIN (MPM_FLAG_NAN for a
// non-finite coordinate) ORed into *bad; key = instance << (block bits + 2d)
// | linear owner block << 2d | local cell of the base node.
template <int DIM>
__device__ __forceinline__ uint32_t bin_key(const DevParams& P, const float* xv, uint32_t inst, unsigned* bad) {
    int b[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        double f = floor(index_arg(xv[a], P.inv_dx));
        if (!(f == f)) {
            *bad |= MPM_FLAG_NAN;
            f = 0.0;
        } else if (f < 0.0 || f + 2.0 > (double)P.cells[a]) {
            *bad |= MPM_FLAG_DOMAIN;
            f = fmin(fmax(f, 0.0), (double)(P.cells[a] - 2));
        }
        b[a] = (int)f;
    }
    uint32_t bl, cell;
    if (DIM == 3) {
        bl = ((uint32_t)(b[2] >> 2) * (uint32_t)P.nblk[1] + (uint32_t)(b[1] >> 2)) * (uint32_t)P.nblk[0] +
             (uint32_t)(b[0] >> 2);
        cell = (b[0] & 3) | ((b[1] & 3) << 2) | ((b[2] & 3) << 4);
    } else {
        bl = (uint32_t)(b[1] >> 2) * (uint32_t)P.nblk[0] + (uint32_t)(b[0] >> 2);
        cell = (b[0] & 3) | ((b[1] & 3) << 2);
    }
    return (inst << (P.blk_bits + 2 * DIM)) | (bl << (2 * DIM)) | cell;
}

template <int DIM>
__device__ __forceinline__ void linear_to_block(const DevParams& P, uint32_t bl, int* bc) {
    bc[0] = (int)(bl % (uint32_t)P.nblk[0]);
    uint32_t r = bl / (uint32_t)P.nblk[0];
    if (DIM == 3) {
        bc[1] = (int)(r % (uint32_t)P.nblk[1]);
        bc[2] = (int)(r / (uint32_t)P.nblk[1]);
    } else {
        bc[1] = (int)r;
        bc[2] = 0;
    }
}

// Block coordinates (and instance) of compact block b (sparse: from its packed
// key; dense: b is the linear block index).
template <int DIM>
__device__ __forceinline__ void block_coords(const DevParams& P, int b, int* bc, int* inst = nullptr) {
    int i = 0;
    if (P.dense)
        linear_to_block<DIM>(P, (uint32_t)b, bc);
    else
        unblock_key<DIM>(P, P.b_keys[b], bc, &i);
    if (inst) *inst = i;
}

// Material of an instance (a single simulation reads the scalar fields).
__device__ __forceinline__ InstMat material(const DevParams& P, int inst) {
    if (P.n_inst > 1) return P.inst[inst];
    InstMat m;
    m.mu = P.mu;
    m.lam = P.lam;
    m.alpha = P.alpha;
    m.dp_coef = P.dp_coef;
    m.dt = P.dt;
    m.p_mass = P.p_mass;
    m.p_vol0 = P.p_vol0;
    m.E = P.E;
    m.dalpha_dphi = P.dalpha_dphi;
    return m;
}

// Compact index of block key K in the block hash table (Eqs. 23-25), -1 if
// the key has no slot or its block did not fit the capacity.
// The slot's value is loaded beside its key, so a hit costs one round trip.
__device__ __forceinline__ int hash_lookup(const DevParams& P, uint64_t K) {
    unsigned s = (unsigned)mix64(K) & P.h_mask_bits;
    for (int r = 0; r < P.n_probe; ++r) {
        const uint64_t cur = P.h_keys[s];
        int val = P.h_vals[s];
        asm volatile("" : "+v"(val));  // keeps the load beside the key's, not behind the compare
        if (cur == K) return val;
        if (cur == EMPTY_KEY) return -1;
        s = (s + 1) & P.h_mask_bits;
    }
    return -1;
}

__device__ __forceinline__ unsigned long long wave_ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ uint64_t wave_or64(uint64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane) {
    unsigned lo = __builtin_amdgcn_readlane((unsigned)v, lane);
    unsigned hi = __builtin_amdgcn_readlane((unsigned)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ int readlane32(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ void raise_flag(DevCounters* c, unsigned f) { atomicOr(&c->flags, f); }

// Inclusive scan across a wave64.
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        unsigned t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan across a 256-thread workgroup; lds needs 4 entries.
__device__ __forceinline__ unsigned wg_excl_scan(unsigned v, unsigned* lds, unsigned* total) {
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    unsigned inc = wave_incl_scan(v);
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    unsigned off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < WG / 64; ++i) {
        unsigned s = lds[i];
        off += (i < w) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// For a pass over tiles whose sums are partials[0 .. tiles): the sum of the
// tiles before `tile` (its exclusive offset) and the sum of all of them, both
// computed by the whole 256-thread workgroup (each workgroup reads the few
// tile sums itself instead of waiting for a separate scan of them).
__device__ __forceinline__ void tile_offset(const unsigned* __restrict__ partials, int tile, int tiles,
                                            unsigned* lds, unsigned* before, unsigned* total) {
    unsigned b = 0, t = 0;
    for (int i = threadIdx.x; i < tiles; i += WG) {
        const unsigned v = partials[i];
        t += v;
        b += i < tile ? v : 0u;
    }
    wg_excl_scan(b, lds, before);
    wg_excl_scan(t, lds, total);
}

// Scan-based construction (scanbuild.hip): the mask domain (bounding box of the
// owner blocks grown by one block on each upper side), written on the device.
struct SbBox {
    int lo[3], hi[3];  // owner-block bounds (lo = INT_MAX, hi = -1 while empty)
    int ext[3];        // extents of the mask domain
    int m;             // its volume in blocks (0: no particle, or above max_m)
    int too_big;       // the volume exceeded max_m
    unsigned total;    // active blocks (sum of the flags)
    int pad[2];
};

// Scratch of the scan-based construction, carved from one allocation: box
// header, the bounding-box partials of the SB_BBOX_WGS workgroups of its pass,
// occupancy (u64), flags and Phi (u32) for up to max_m blocks of the domain,
// scan partials; owner segment bounds (step build only, may be null).
constexpr int SB_BBOX_WGS = 1024;
constexpr size_t sb_scratch_size(long long max_m) {
    return 256 + (size_t)SB_BBOX_WGS * 8 * sizeof(int) + (size_t)max_m * (8 + 4 + 4) +
           (size_t)((max_m + SCAN_TILE - 1) / SCAN_TILE + 1) * sizeof(unsigned) + 256;
}
struct SbScratch {
    SbBox* box;
    int* bbp;  // per workgroup of the bounding-box pass: lo[3], hi[3]
    uint64_t* occ;
    unsigned* flag;
    unsigned* phi;
    unsigned* partials;
    int* seg_lo;
    int* seg_hi;
    long long max_m;
};

// Work items of a block holding cnt particles (none for a block that only
// holds stencil nodes).
__device__ __forceinline__ unsigned block_chunks(const DevParams& P, int cnt) {
    return cnt > 0 ? (unsigned)((cnt + P.chunk - 1) / P.chunk) : 0u;
}

// Box [lo, hi] over the workgroup's threads, left in every thread.
__device__ __forceinline__ void box_reduce(int* lo, int* hi, int (*red)[6]) {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int m = 32; m >= 1; m >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], m));
            hi[a] = max(hi[a], __shfl_xor(hi[a], m));
        }
        if (__lane_id() == 0) {
            red[w][a] = lo[a];
            red[w][3 + a] = hi[a];
        }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int q = 0; q < WG / 64; ++q) {
            lo[a] = min(lo[a], red[q][a]);
            hi[a] = max(hi[a], red[q][3 + a]);
        }
}

// ---------------------------------------------------------------------------
// host-side launchers (each returns hipError_t of the launch)
hipError_t scan_exclusive(const unsigned* in, unsigned* out, int n, const int* n_dev, unsigned* partials,
                          unsigned* total_out, hipStream_t s);
int scan_partials_size(int n);
hipError_t launch_tile_sums(const DevParams& P, int tiles, hipStream_t s);
size_t sb_scratch_bytes(long long max_m);
SbScratch sb_carve(void* base, long long max_m, int* seg_lo, int* seg_hi);
hipError_t launch_scan_active(const DevParams& P, const float* x, int n, const SbScratch& S, uint64_t* keys_out,
                              uint64_t* masks_out, int cap, hipStream_t s);
hipError_t launch_build_scan(const DevParams& P, const uint32_t* skeys, int n, const SbScratch& S,
                             unsigned* partials, hipStream_t s);
hipError_t launch_work_items(const DevParams& P, unsigned* partials, hipStream_t s);
long long scan_active_static_max_blocks();
hipError_t launch_scan_active_static(const DevParams& P, const float* x, int n, uint64_t* keys_out,
                                     uint64_t* masks_out, int cap, SbBox* box_host, hipStream_t s);

hipError_t radix_sort(const uint32_t* keys_in, uint32_t* k0, uint32_t* k1, uint32_t* v0, uint32_t* v1, int n,
                      int key_bits, unsigned* hist, unsigned* partials, uint32_t** keys_out, uint32_t** vals_out,
                      hipStream_t s);
int radix_hist_size(int n);
// Passes of the sort; the sorted keys end in k0 when the count is odd, else in k1.
constexpr int radix_passes(int key_bits) { return key_bits <= 8 ? 1 : (key_bits + 7) / 8; }

// Full sort by counting in a table of owner blocks (tabsort.hip).  Builds of
// 4,096 / 262,144 / 2,097,152 / 4,194,304 particles (439,000 owner blocks in the
// domain) that were in order, as every step after the first finds them: 29 / 32 /
// 68 / 109 us, by radix passes 96 / 122 / 165 / 221; in random order 30 / 71 /
// 228 / 397, by radix passes 96 / 123 / 165 / 222 (the two lines cross at 1.2
// million; all with 8 particles per cell).  So a context that sorts in every step takes the table, one that
// sorts only for its first build takes it up to TAB_MAX_ONCE particles.
// Largest domain: 32 MB of counts and positions; 4.1 million blocks add 10 us.
constexpr int TAB_MAX_IDS = 1 << 22;
constexpr int TAB_MAX_ONCE = 1 << 20;
// Entries per thread of the scan over the table.  Its tiles are all the
// parallelism it has (12 tiles of 2048 in the domain of 262,144 particles, a
// dense grid's block tables written by each thread in turn: 9 us; of 512: 5),
// and every tile reads the sums of all.  Builds of 262,144 particles with 2 / 8
// entries: 17,576 blocks hashed 33.8 / 34.5 us, dense 29.7 / 35.4; 250,047 34.7 /
// 34.8 and 59.4 / 63.6; 438,976 hashed 35.6 / 34.8; 1,061,208 40.1 / 36.6.
constexpr int TAB_SMALL_IDS = 1 << 18;
constexpr int TAB_SMALL_ITEMS = 2;
constexpr int tab_items(long long ids, bool scan_build) {
    return !scan_build && ids <= TAB_SMALL_IDS ? TAB_SMALL_ITEMS : SCAN_ITEMS;
}
// Particles of a block that a workgroup puts in order in LDS (5 bytes each): up to
// TAB_BATCH they are held in registers meanwhile; up to TAB_STAGE as many
// workgroups stay resident as the wave slots take; contexts whose full cells hold
// more (half as many again as at rest still fit) stage up to TAB_STAGE_MAX.  What
// does not fit is ordered by one wave in passes over global memory.
// Above TAB_MAX_PER_CELL particles in a cell at rest the order within a cell, which
// each particle finds by counting the smaller indices of its cell, costs more
// than the radix passes, above TAB_MAX_PER_BLOCK in a block the two readings do, and
// those contexts keep the radix sort.  Full steps of 262,144 particles with 8 / 27 / 64 / 125 per cell by the table 75 / 107 / 198 / 467
// us, by radix passes 162 / 164 / 200 / 318 (with blocks of more than 1024
// particles left to one wave 75 / 193 / 335 / 632); 2D with 16 / 64 / 100 / 144 per
// cell 75 / 126 / 145 / 206, radix 118 / 147 / 149 / 175, on a dense grid 55 / 111 /
// 137 / 199 and 95 / 132 / 163 / 169; 2.1 million with 27 per cell 290 (308 staging
// 8192), radix 360.
// Blocks of up to TAB_WAVE particles are ordered by a wave each where a block at rest
// holds TAB_WAVE_MEAN or fewer: full steps of 4 million particles in 2D with 4 per cell
// (64 in a block) 516 us, a workgroup each 644, the radix sort 597; 16,641 with 9 per
// cell (144) 47.6 by waves and 45.9 by workgroups.
constexpr int TAB_WAVE = 128, TAB_WAVE_MEAN = 96;
constexpr int TAB_BATCH = 1024, TAB_STAGE = 3072, TAB_STAGE_MAX = 8192;
constexpr double TAB_MAX_PER_CELL = 110.0, TAB_MAX_PER_BLOCK = 4608.0;
struct TabSort {
    unsigned* cnt;    // particles per owner block (instance and linear block); zero between sorts
    unsigned* start;  // first position of each occupied block
    uint4* ent;       // occupied blocks in ascending order: block, first position, particles
    unsigned* part;   // tile sums of the scan: particles, occupied blocks, work items (4 words per tile;
                      // 8 for a scan-built context, whose build keeps its own there afterwards)
    int* n_ent;
    int ids, ent_cap;
    int stage;  // particles of a block that fit LDS: TAB_STAGE or TAB_STAGE_MAX
    bool waves;  // small blocks: a wave each
    // scan-built contexts: occupied base cells and entry of each block (occ zero
    // between builds), bounding box of each tile's occupied blocks
    uint64_t* occ;
    int* eidx;
    int* box;  // 8 words per tile: lo[3], -, hi[3], -
};
enum TabMode {
    TAB_HASH,   // the sort clears the block hash and inserts every block
    TAB_DENSE,  // the sort fills a dense grid's block tables and work items
    TAB_SCAN    // the sort leaves counts and occupied cells for launch_build_scan_tab
};
hipError_t launch_tab_init(const TabSort& T, hipStream_t s);
// keys: unsorted; rank, tmp: scratch; order, skeys: the result (skeys may be tmp).
hipError_t launch_tab_sort(const DevParams& P, const TabSort& T, const uint32_t* keys, uint32_t* rank, uint32_t* tmp,
                           uint32_t* order, uint32_t* skeys, int n, unsigned H, TabMode mode, hipStream_t s);
hipError_t launch_build_scan_tab(const DevParams& P, const TabSort& T, const SbScratch& S, hipStream_t s);

hipError_t launch_bin(const DevParams& P, const float* x, const uint32_t* inst, int n, uint32_t* keys, hipStream_t s);
// The sorted keys are not written (after an incremental re-sort nothing reads
// them; P2G takes the cell ranges from the re-sort's per-entry table).  movers
// and tgt: n entries each (the movers of each work item, listed from the item's
// first position on, and each mover's target, which the route records for the
// placement).  Fills the block hash as well.
hipError_t launch_resort(const DevParams& P, const uint32_t* keys_new, uint32_t* vals_out, uint32_t* movers,
                         uint32_t* tgt, int n, unsigned H, unsigned* partials, hipStream_t s, bool counted = false);
hipError_t launch_resort_init(const DevParams& P, unsigned H, hipStream_t s);
// Buffers of the ascending-key Phi order (MPM_FLAG_DETERMINISTIC_ORDER): block
// tables in slot order, the slot of each, and a radix sort of block_cap
// entries (keys, values, histograms).
struct DetTables {
    uint64_t* keys;
    uint64_t* mask;
    int* start;
    int* count;
    int* slot;
    uint32_t* k[2];
    uint32_t* v[2];
    unsigned* hist;
};
// inserted: the re-sort has filled the block hash already.
hipError_t launch_build_sparse(const DevParams& P, const uint32_t* skeys, int n, unsigned H, unsigned* partials,
                               hipStream_t s, bool inserted = false, const DetTables* det = nullptr);
hipError_t launch_build_dense(const DevParams& P, const uint32_t* skeys, int n, int n_blocks, unsigned* partials,
                              hipStream_t s);
hipError_t launch_dense_neighbours(const DevParams& P, int n_blocks, hipStream_t s);
hipError_t launch_grid_clear(const DevParams& P, int n_blocks, hipStream_t s);
// P2G's second pass (sparse grids): the sums of the tiles; with the grid update
// (Eqs. 8-12), which leaves velocities instead of momenta in the grid; or none,
// where G2P forms the nodes it reads (launch_g2p with gather) and nothing else
// reads the grid.
enum P2GSecond { P2G_SUM, P2G_UPDATE, P2G_LEFT_TO_G2P };
hipError_t launch_p2g(const DevParams& P, const float* x, const float* v, const float* C, const float* tau, int n,
                      const uint32_t* order, const uint32_t* skeys, uint32_t* osrc, int grid_blocks, hipStream_t s,
                      P2GSecond second = P2G_SUM);
hipError_t launch_grid_update(const DevParams& P, long long n_nodes_host, int grid_blocks, hipStream_t s);
hipError_t launch_g2p(const DevParams& P, const float* x_in, const float* F_in, const uint32_t* id_in,
                      const uint32_t* inst_in, float* x_out, float* v_out, float* C_out, float* F_out, float* tau_out,
                      uint32_t* id_out, uint32_t* inst_out, int n, const uint32_t* osrc, int block_size,
                      int grid_blocks, hipStream_t s, uint32_t* keys_out = nullptr,
                      uint32_t* movers_out = nullptr, bool gather = false);
hipError_t launch_clear_flags(DevCounters* c, hipStream_t s);
// Reverse kernels; osrc[o]: input index of the particle at G2P output position o.
constexpr int ADJ_MAX_WGS = 8192;  // workgroups of the per-particle kernels at most
hipError_t launch_g2p_adj(const DevParams& P, const float* x, const float* F, const float* const* out_bar, float* x_bar,
                          float* F_bar, int n, const uint32_t* osrc, hipStream_t s);
hipError_t launch_scatter_adj(const DevParams& P, int n, const uint32_t* skeys, int grid_blocks, hipStream_t s);
hipError_t launch_grid_adj(const DevParams& P, hipStream_t s);
hipError_t launch_p2g_adj(const DevParams& P, const float* const* in, float* const* in_bar, int n,
                          const uint32_t* osrc, hipStream_t s);
hipError_t launch_copy_active(const DevParams& P, uint64_t* keys, uint64_t* masks, int cap, hipStream_t s);

}  // namespace mpmx
