// Active-node indexing on the GPU (Methods 3.3, Algorithms 5-6; Eqs. 22-25).
//
//   k_bin           base node per particle (float64 index arithmetic), owner
//                   block and a u32 sort key = linear block id << 2d | local
//                   cell of the base node;
//   sort            groups particles by owner block: the counting sort of
//                   tabsort.hip (in large domains the radix sort of sort.hip),
//                   or after a build of as many particles the incremental
//                   re-sort of resort.hip;
//   k_hash_clear    keys <- EMPTY, masks <- 0 (Algorithm 5, initialisation);
//   k_hash_insert   per sorted particle: the stencil touches its owner block and
//                   only the upper neighbours it spills into (base local index
//                   >= 2 on an axis), so at most 2^d blocks.  Lanes of a wave64
//                   that share an owner block are merged (ballot/readlane loop)
//                   and their node masks OR-reduced, then one lane per touched
//                   block claims or finds the slot: packed key (Eq. 22), mixer
//                   (Eq. 23), slot h & (H - 1) (Eq. 24), linear probing (Eq. 25)
//                   with a compare-and-swap on EMPTY (Algorithm 6), and ORs the
//                   node mask into the slot.  The owner run boundaries of the
//                   sorted order are recorded per slot.
//   (the counting sort clears and fills the hash table itself, an occupied
//   block at a time; so does the incremental re-sort, per entry)
//   compaction      prefix sums over the occupied slots (counted per tile of the
//                   table by the insertion) -> Phi in slot order; block keys,
//                   masks and owner segments in Phi order; overflow when more
//                   than block_capacity slots are occupied (the counter check
//                   of Algorithm 6); the same pass numbers the work items
//                   (owner segments in chunks) in Phi order and writes them,
//                   except for the key-ordered Phi, whose items follow from a
//                   scan of per-block counts after the reordering.  It also
//                   prepares the counting of the next incremental re-sort.
//   neighbours      the insertion of an owner block records the slots of the
//                   blocks its stencils reach; P2G, when every Phi is known,
//                   makes the neighbour tables from them, so nothing probes the
//                   table a second time.  (The dense baseline also clears its
//                   grid; the sparse P2G writes every node of every active
//                   block.)
#include "hash.h"
#include "internal.h"

namespace mpmx {

constexpr int BIN_PER_THREAD = 2;  // particles per thread of k_bin (loads issued together)

template <int DIM>
__global__ __launch_bounds__(WG) void k_bin(DevParams P, const float* __restrict__ x,
                                            const uint32_t* __restrict__ inst, int n, uint32_t* __restrict__ keys) {
    const int i0 = blockIdx.x * WG * BIN_PER_THREAD + threadIdx.x;
    if (P.rs_tile && blockIdx.x == 0) {
        // a separate binning pass precedes a re-sort's own counting: drop what
        // a G2P may have counted for a build that did not follow
        for (int t = threadIdx.x; t < (P.block_cap + RS_TILE - 1) / RS_TILE; t += WG) P.rs_tile[t * LINE] = 0u;
    }
    float xv[BIN_PER_THREAD][3];
    uint32_t iv[BIN_PER_THREAD];
#pragma unroll
    for (int k = 0; k < BIN_PER_THREAD; ++k) {
        const int i = i0 + k * WG;
        iv[k] = 0u;
#pragma unroll
        for (int a = 0; a < 3; ++a) xv[k][a] = 0.f;
        if (i < n) {
#pragma unroll
            for (int a = 0; a < DIM; ++a) xv[k][a] = x[(size_t)a * n + i];
            if (P.n_inst > 1 && inst) iv[k] = inst[i];
        }
    }
    unsigned bad = 0;
#pragma unroll
    for (int k = 0; k < BIN_PER_THREAD; ++k) {
        const int i = i0 + k * WG;
        if (i >= n) break;
        uint32_t in = iv[k];
        if (in >= (uint32_t)max(P.n_inst, 1)) {
            bad |= MPM_FLAG_DOMAIN;
            in = (uint32_t)max(P.n_inst, 1) - 1;
        }
        keys[i] = bin_key<DIM>(P, xv[k], in, &bad);
    }
    if (bad) raise_flag(P.ctr, bad);
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_hash_clear(DevParams P, unsigned H) {
    clear_hash<1 << DIM, true>(P, H, blockIdx.x * WG + threadIdx.x, gridDim.x * WG);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        P.ctr->nb = 0;
        P.ctr->n_touched = 0;
        P.ctr->n_work = 0;
    }
}

constexpr int HI_ROUNDS = 4;  // sorted particles per lane of k_hash_insert (a wave covers 256)

// Sorted particles in runs of 256 per wave.  A run of equal owner blocks is one
// group; a group that continues from the previous round of the same wave is
// merged, so each wave inserts each of its owner blocks once.  Per group: the
// OR of its base-cell bits, the node masks of the owner and its 2^d - 1 upper
// neighbours by bit dilation, one insert per touched block (lane d takes
// neighbour d), and the owner segment's first / one-past-last sorted position
// where the segment starts / ends inside this wave.
template <int DIM>
__global__ __launch_bounds__(WG) void k_hash_insert(DevParams P, const uint32_t* __restrict__ skeys, int n) {
    constexpr int NB = 1 << DIM;
    constexpr int CB = 2 * DIM;
    const int lane = __lane_id();
    const int base = ((blockIdx.x * WG + (int)threadIdx.x) >> 6) * 64 * HI_ROUNDS;
    if (base >= n) return;  // whole wave
    const int stop = min(base + 64 * HI_ROUNDS, n);
    // owner segments (instance and block) just before and after this wave's range
    const uint32_t seg_before = base > 0 ? (skeys[base - 1] >> CB) : ~0u;
    const uint32_t seg_after = stop < n ? (skeys[stop] >> CB) : ~0u;
    uint32_t key[HI_ROUNDS];
#pragma unroll
    for (int r = 0; r < HI_ROUNDS; ++r) {
        const int i = base + r * 64 + lane;
        key[r] = i < n ? skeys[i] : 0u;
    }
    bool have = false;
    uint32_t p_seg = 0;
    uint64_t p_occ = 0;
    int p_first = 0, p_end = 0;
    auto flush = [&]() {
        const int slot = lane < NB ? insert_block<DIM>(P, p_seg, p_occ, lane) : -1;
        const int own = readlane32(slot, 0);  // lane 0 holds the owner block
        // a block that spans waves is inserted by each with a part of its
        // cells: every part records the slots it reached
        if (own >= 0 && slot >= 0) P.h_nslot[(size_t)own * NB + lane] = slot;
        if (lane == 0 && own >= 0) {
            if (p_first > base || seg_before != p_seg) P.h_start[own] = p_first;
            if (p_end < stop || seg_after != p_seg) P.h_end[own] = p_end;
        }
    };
#pragma unroll
    for (int r = 0; r < HI_ROUNDS; ++r) {
        const int i = base + r * 64 + lane;
        const bool valid = i < n;
        const uint32_t seg = key[r] >> CB;
        const uint32_t cell = key[r] & ((1u << CB) - 1u);
        unsigned long long todo = __ballot(valid);
        while (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const uint32_t g = (uint32_t)readlane32((int)seg, leader);
            const bool mine = valid && seg == g;
            const unsigned long long grp = __ballot(mine);
            const uint64_t occ = readlane64(wave_or64(mine ? (1ull << cell) : 0ull), leader);
            const int first = base + r * 64 + leader;
            const int last = base + r * 64 + (63 - __clzll((long long)grp));
            if (have && g == p_seg) {
                p_occ |= occ;
                p_end = last + 1;
            } else {
                if (have) flush();
                have = true;
                p_seg = g;
                p_occ = occ;
                p_first = first;
                p_end = last + 1;
            }
            todo &= ~grp;
        }
    }
    if (have) flush();
}

// Work items per tile of the table (after k_hash_insert, whose waves see only
// parts of a block; a re-sort's insertion counts them itself).
__global__ __launch_bounds__(WG) void k_count_items(DevParams P, int H) {
    __shared__ unsigned lds[WG / 64];
    const int base = blockIdx.x * SCAN_TILE + threadIdx.x;
    int st[SCAN_ITEMS], en[SCAN_ITEMS];
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        const int idx = min(base + j * WG, H - 1);
        st[j] = P.h_start[idx];
        en[j] = P.h_end[idx];
    }
    unsigned w = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) w += base + j * WG < H && st[j] >= 0 ? block_chunks(P, en[j] - st[j]) : 0u;
    unsigned tot;
    wg_excl_scan(w, lds, &tot);
    if (threadIdx.x == 0) P.t_cnt[blockIdx.x * LINE + 1] = tot;
}

// Compaction: Phi in slot order and the block tables, one workgroup per tile of
// SCAN_TILE slots, whose occupied slots and work items the insertion counted
// (t_cnt), so that each tile adds up the counts before it and no pass over the
// table precedes this one.  A table is a few per cent full: the tile's occupied
// slots are first listed in LDS (64 contiguous keys per wave and round, a
// ballot and a popcount each), then every thread takes one slot of the list.
// The passes are bound by latency, not bandwidth.  (With eight slots per
// thread carried through, and the counting as a pass of its own, the two took
// 4.8 + 10.2 us at 32,768 slots and 8.8 + 17.6 us at 2,097,152.)
// ITEMS: also the work items and the state that the counting of the next
// incremental re-sort starts from.
// PRE: the sums over the tiles have been made (launch_tile_sums).
template <int DIM, bool ITEMS, bool PRE>
__global__ __launch_bounds__(WG) void k_compact_write(DevParams P, int H, int tiles) {
    constexpr int NB = 1 << DIM, NC = 1 << (2 * DIM);
    constexpr int NW = WG / 64, ROUNDS = SCAN_TILE / WG;
    __shared__ unsigned short list[SCAN_TILE];  // occupied slots of the tile, ascending
    __shared__ unsigned red[NW][4], wcnt[NW * ROUNDS], lds[NW];
    const int lane = __lane_id(), wv = threadIdx.x >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int base = blockIdx.x * SCAN_TILE;
    uint64_t k[ROUNDS];
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int idx = base + j * WG + (int)threadIdx.x;
        k[j] = idx < H ? P.h_keys[idx] : EMPTY_KEY;
    }
    // sums over the tiles: occupied slots and items before this one, and all
    unsigned sum[4] = {0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; !PRE && i < tiles; i += WG) {
        const unsigned c = P.t_cnt[i * LINE], it = P.t_cnt[i * LINE + 1];
        sum[0] += i < (int)blockIdx.x ? c : 0u;
        sum[1] += i < (int)blockIdx.x ? it : 0u;
        sum[2] += c;
        sum[3] += it;
    }
    unsigned long long occ[ROUNDS];
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        occ[j] = __ballot(k[j] != EMPTY_KEY);
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
    // every wave scans the NW * ROUNDS ballot counts for itself
    const unsigned mine = lane < NW * ROUNDS ? wcnt[lane] : 0u;
    const unsigned inc = wave_incl_scan(mine);
    const int n_occ = readlane32((int)inc, 63);
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int q = j * NW + wv;
        const unsigned first = (unsigned)__shfl((int)(inc - mine), q);
        if (k[j] != EMPTY_KEY) list[first + (unsigned)__popcll(occ[j] & lt)] = (unsigned short)(j * WG + threadIdx.x);
    }
    __syncthreads();
    unsigned phi0 = 0, it0 = 0, total = 0, wtotal = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        phi0 += red[q][0];
        it0 += red[q][1];
        total += red[q][2];
        wtotal += red[q][3];
    }
    if (PRE) {
        phi0 = P.t_cnt[(size_t)blockIdx.x * LINE + 2];
        it0 = P.t_cnt[(size_t)blockIdx.x * LINE + 3];
        total = P.t_cnt[(size_t)tiles * LINE + 2];
        wtotal = P.t_cnt[(size_t)tiles * LINE + 3];
    }
    bool over = false;
#pragma unroll 1
    for (int t0 = 0; t0 < n_occ; t0 += WG) {
        const bool o = t0 + (int)threadIdx.x < n_occ;
        const int idx = o ? base + list[t0 + threadIdx.x] : 0;
        const unsigned phi = phi0 + (unsigned)(t0 + (int)threadIdx.x);
        uint64_t key = 0, mask = 0;
        int st = -1, en = -1, ent = -1;
        if (o) {
            key = P.h_keys[idx];
            mask = P.h_mask[idx];
            st = P.h_start[idx];
            en = P.h_end[idx];
            if (P.b_entry) ent = P.h_entry[idx];
        }
        const int cnt = st >= 0 ? en - st : 0;
        const unsigned chunks = block_chunks(P, cnt);
        unsigned w = it0;
        if (ITEMS) {
            unsigned tot;
            w += wg_excl_scan(chunks, lds, &tot);
            it0 += tot;
        }
        const bool fits = o && phi < (unsigned)P.block_cap;
        if (fits) {
            P.b_keys[phi] = key;
            P.b_mask[phi] = mask;
            P.b_start[phi] = st;
            P.b_count[phi] = cnt;
            P.h_vals[idx] = (int)phi;
            P.b_hs[phi] = idx;
            if (ITEMS) {
                if (P.b_entry) P.b_entry[phi] = ent;
                P.b_chunks[phi] = chunks;
                P.b_chunk_off[phi] = w;
#pragma unroll
                for (int d = 0; d < NB; d += 4)  // set by the P2G of the blocks that reach this one
                    *(int4*)&P.b_lo[(size_t)phi * NB + d] = make_int4(-1, -1, -1, -1);
                for (unsigned q = 0; q < chunks; ++q) {
                    if (w + q >= (unsigned)P.work_cap) {
                        over = true;
                        break;
                    }
                    P.w_block[w + q] = (int)phi;
                    P.w_start[w + q] = st + (int)q * P.chunk;
                    P.w_end[w + q] = min(st + ((int)q + 1) * P.chunk, en);
                }
            }
        } else if (o) {
            P.h_vals[idx] = -1;
            over = true;
        }
        if (ITEMS && P.rs_stay) {
            // for the next incremental re-sort, when a G2P counts for it: the
            // owner part of the block's sort key, and cleared counts where G2P
            // will not store them whole (no particle, or several work items
            // adding theirs; the cell counts of a block without particles are
            // not read)
            if (fits) {
                int bc[3], inst;
                unblock_key<DIM>(P, key, bc, &inst);
                bool in_range = inst < max(P.n_inst, 1);
#pragma unroll
                for (int a = 0; a < DIM; ++a) in_range = in_range && bc[a] >= 0 && bc[a] < P.nblk[a];
                const uint32_t bl = DIM == 3 ? ((uint32_t)bc[2] * (uint32_t)P.nblk[1] + (uint32_t)bc[1]) *
                                                       (uint32_t)P.nblk[0] + (uint32_t)bc[0]
                                             : (uint32_t)bc[1] * (uint32_t)P.nblk[0] + (uint32_t)bc[0];
                P.rs_oldblk[phi] = in_range ? ((uint32_t)inst << P.blk_bits) | bl : ~0u;
                if (chunks != 1u || total > (unsigned)P.block_cap) P.rs_cnt[phi] = 0u;  // past the capacity no G2P counts
            }
            unsigned long long multi = __ballot(fits && chunks > 1u);
            while (multi) {  // a row per step, contiguous
                const int l = __ffsll((long long)multi) - 1;
                const unsigned p = (unsigned)readlane32((int)phi, l);
                if (lane < NC) P.rs_stay[(size_t)p * NC + lane] = 0u;
                multi &= multi - 1ull;
            }
        }
    }
    if (over) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            P.ctr->n_touched = total;
            P.ctr->nb = min((int)total, P.block_cap);
            if (ITEMS) {
                // items of blocks past the capacity were not written: no work then
                P.ctr->n_work = total <= (unsigned)P.block_cap ? (int)wtotal : 0;
                P.ctr->rs_n_new = 0;    // the new blocks the next re-sort's route claims
                P.ctr->rs_new_pos = 0;  // and their particles
            }
        }
        if (ITEMS && P.rs_tile)
            for (int t = threadIdx.x; t < (P.block_cap + RS_TILE - 1) / RS_TILE; t += WG) P.rs_tile[t * LINE] = 0u;
    }
}

// Ascending-key order of Phi (MPM_FLAG_DETERMINISTIC_ORDER).  The compaction
// wrote the block tables in slot order into the alternate arrays; the blocks
// are sorted by their coordinates (instance, i, j, k), which is the order of
// the Eq. 22 keys, and gathered into the block tables in that order.
template <int DIM>
__global__ __launch_bounds__(WG) void k_det_keys(DevParams P, const uint64_t* __restrict__ alt_keys,
                                                 uint32_t* __restrict__ rank_keys, uint32_t sentinel) {
    const int nb = P.ctr->nb;
    for (int b = blockIdx.x * WG + threadIdx.x; b < P.block_cap; b += gridDim.x * WG) {
        uint32_t r = sentinel;
        if (b < nb) {
            int bc[3], inst;
            unblock_key<DIM>(P, alt_keys[b], bc, &inst);
            const uint32_t lin = DIM == 3 ? ((uint32_t)bc[0] * (uint32_t)P.nblk[1] + (uint32_t)bc[1]) *
                                                    (uint32_t)P.nblk[2] + (uint32_t)bc[2]
                                          : (uint32_t)bc[0] * (uint32_t)P.nblk[1] + (uint32_t)bc[1];
            r = ((uint32_t)inst << P.blk_bits) | lin;
        }
        rank_keys[b] = r;
    }
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_det_apply(DevParams P, DetTables T, const uint32_t* __restrict__ sorted) {
    constexpr int NB = 1 << DIM;
    const int nb = P.ctr->nb;
    for (int r = blockIdx.x * WG + threadIdx.x; r < nb; r += gridDim.x * WG) {
        const int b = (int)sorted[r];
        P.b_keys[r] = T.keys[b];
        P.b_mask[r] = T.mask[b];
        P.b_start[r] = T.start[b];
        const int cnt = T.count[b], slot = T.slot[b];
        P.b_count[r] = cnt;
        P.b_chunks[r] = block_chunks(P, cnt);
        P.h_vals[slot] = r;
#pragma unroll
        for (int d = 0; d < NB; ++d) P.b_lo[(size_t)r * NB + d] = -1;
        P.b_hs[r] = slot;
    }
}

__global__ __launch_bounds__(WG) void k_work_write(DevParams P) {
    const int nb = P.ctr->nb;
    bool over = false;
    for (int b = blockIdx.x * WG + threadIdx.x; b < nb; b += gridDim.x * WG) {
        const int c = (int)P.b_chunks[b];
        const int off = (int)P.b_chunk_off[b];
        const int st = P.b_start[b], cnt = P.b_count[b];
        for (int j = 0; j < c; ++j) {
            const int w = off + j;
            if (w >= P.work_cap) {
                over = true;
                break;
            }
            P.w_block[w] = b;
            P.w_start[w] = st + j * P.chunk;
            P.w_end[w] = min(st + (j + 1) * P.chunk, st + cnt);
        }
    }
    if (over) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_grid_clear(DevParams P, long long n_nodes) {
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (long long s = (long long)blockIdx.x * WG + threadIdx.x; s < n_nodes; s += (long long)gridDim.x * WG)
        P.grid[s] = z;
}

// ---- dense baseline: Phi(b) = linear block index over the whole domain ----
__global__ __launch_bounds__(WG) void k_dense_clear_seg(DevParams P, int n_blocks) {
    for (int b = blockIdx.x * WG + threadIdx.x; b < n_blocks; b += gridDim.x * WG) {
        P.b_start[b] = -1;
        P.b_count[b] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        P.ctr->nb = n_blocks;
        P.ctr->n_touched = n_blocks;
        P.ctr->n_work = 0;
    }
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_dense_segments(DevParams P, const uint32_t* __restrict__ skeys, int n) {
    constexpr int CB = 2 * DIM;
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i >= n) return;
    const uint32_t bl = skeys[i] >> CB;
    if (i == 0 || (skeys[i - 1] >> CB) != bl) P.b_start[bl] = i;
    if (i == n - 1 || (skeys[i + 1] >> CB) != bl) P.b_count[bl] = i + 1;  // end, converted below
}

__global__ __launch_bounds__(WG) void k_dense_counts(DevParams P, int n_blocks) {
    for (int b = blockIdx.x * WG + threadIdx.x; b < n_blocks; b += gridDim.x * WG) {
        const int st = P.b_start[b];
        const int cnt = st >= 0 ? P.b_count[b] - st : 0;
        P.b_count[b] = cnt;
        P.b_chunks[b] = block_chunks(P, cnt);
    }
}

// Upper neighbours on a dense grid: the same for every build, written once.
template <int DIM>
__global__ __launch_bounds__(WG) void k_dense_neighbours(DevParams P, int n_blocks) {
    constexpr int NB = 1 << DIM;
    for (int b = blockIdx.x * WG + threadIdx.x; b < n_blocks; b += gridDim.x * WG) {
        int bc[3];
        linear_to_block<DIM>(P, (uint32_t)b, bc);
#pragma unroll
        for (int d = 0; d < NB; ++d) {
            const int x = bc[0] + (d & 1), y = bc[1] + ((d >> 1) & 1), z = bc[2] + ((d >> 2) & 1);
            const bool in = x < P.nblk[0] && y < P.nblk[1] && (DIM == 2 || z < P.nblk[2]);
            P.b_nbr[(size_t)b * NB + d] = in ? (DIM == 3 ? (z * P.nblk[1] + y) * P.nblk[0] + x : y * P.nblk[0] + x) : -1;
        }
    }
}

__global__ __launch_bounds__(WG) void k_copy_active(DevParams P, uint64_t* keys, uint64_t* masks, int cap) {
    const int nb = min(P.ctr->nb, cap);
    for (int b = blockIdx.x * WG + threadIdx.x; b < nb; b += gridDim.x * WG) {
        keys[b] = P.b_keys[b];
        masks[b] = P.b_mask[b];
    }
}

static int grid_for(long long items, int cap_wgs = 8192) {
    long long g = (items + WG - 1) / WG;
    if (g < 1) g = 1;
    if (g > cap_wgs) g = cap_wgs;
    return (int)g;
}

hipError_t launch_bin(const DevParams& P, const float* x, const uint32_t* inst, int n, uint32_t* keys, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int g = (n + WG * BIN_PER_THREAD - 1) / (WG * BIN_PER_THREAD);
    if (P.dim == 3)
        k_bin<3><<<g, WG, 0, s>>>(P, x, inst, n, keys);
    else
        k_bin<2><<<g, WG, 0, s>>>(P, x, inst, n, keys);
    return hipGetLastError();
}

namespace {
template <int DIM>
hipError_t build_sparse(const DevParams& P, const uint32_t* skeys, int n, unsigned H, unsigned* partials, hipStream_t s,
                        bool inserted, const DetTables* det) {
    const int tiles = ((int)H + SCAN_TILE - 1) / SCAN_TILE;
    if (!inserted) {
        k_hash_clear<DIM><<<grid_for(H), WG, 0, s>>>(P, H);
        if (n > 0) {
            const int per_wg = WG * HI_ROUNDS;
            k_hash_insert<DIM><<<(n + per_wg - 1) / per_wg, WG, 0, s>>>(P, skeys, n);
            if (!det) k_count_items<<<tiles, WG, 0, s>>>(P, (int)H);
        }
    }
    const bool pre = tiles > FOLD_MAX_TILES;
    if (pre) {
        hipError_t e = launch_tile_sums(P, tiles, s);
        if (e != hipSuccess) return e;
    }
    // without the key order, Phi is slot order and the compaction also writes
    // the work items
    if (!det) {
        const auto k = !pre ? k_compact_write<DIM, true, false> : k_compact_write<DIM, true, true>;
        k<<<tiles, WG, 0, s>>>(P, (int)H, tiles);
        // no grid clear: the second P2G pass writes every node of every active block
        return hipGetLastError();
    }
    // compaction in slot order into the alternate tables, then the blocks
    // sorted by key and gathered into the block tables
    const int gb = grid_for(P.block_cap, 2048);
    DevParams Pa = P;
    Pa.b_keys = det->keys;
    Pa.b_mask = det->mask;
    Pa.b_start = det->start;
    Pa.b_count = det->count;
    Pa.b_hs = det->slot;
    const auto k = !pre ? k_compact_write<DIM, false, false> : k_compact_write<DIM, false, true>;
    k<<<tiles, WG, 0, s>>>(Pa, (int)H, tiles);
    const int kb = P.blk_bits + (P.n_inst > 1 ? 6 : 0);
    const uint32_t sentinel = kb >= 32 ? 0xFFFFFFFFu : ((1u << kb) - 1u);
    k_det_keys<DIM><<<gb, WG, 0, s>>>(P, det->keys, det->k[1], sentinel);
    uint32_t *ko = nullptr, *vo = nullptr;
    hipError_t e = radix_sort(det->k[1], det->k[0], det->k[1], det->v[0], det->v[1], P.block_cap, kb, det->hist, partials,
                              &ko, &vo, s);
    if (e != hipSuccess) return e;
    k_det_apply<DIM><<<gb, WG, 0, s>>>(P, *det, vo);
    e = hipGetLastError();
    return e == hipSuccess ? launch_work_items(P, partials, s) : e;
}
}  // namespace

hipError_t launch_build_sparse(const DevParams& P, const uint32_t* skeys, int n, unsigned H, unsigned* partials,
                               hipStream_t s, bool inserted, const DetTables* det) {
    return P.dim == 3 ? build_sparse<3>(P, skeys, n, H, partials, s, inserted, det)
                      : build_sparse<2>(P, skeys, n, H, partials, s, inserted, det);
}

// Work items: exclusive scan of the per-block chunk counts, then the items.
hipError_t launch_work_items(const DevParams& P, unsigned* partials, hipStream_t s) {
    hipError_t e = scan_exclusive(P.b_chunks, P.b_chunk_off, P.block_cap, &P.ctr->nb, partials,
                                  (unsigned*)&P.ctr->n_work, s);
    if (e != hipSuccess) return e;
    k_work_write<<<grid_for(P.block_cap, 2048), WG, 0, s>>>(P);
    return hipGetLastError();
}

hipError_t launch_dense_neighbours(const DevParams& P, int n_blocks, hipStream_t s) {
    if (P.dim == 3)
        k_dense_neighbours<3><<<grid_for(n_blocks), WG, 0, s>>>(P, n_blocks);
    else
        k_dense_neighbours<2><<<grid_for(n_blocks), WG, 0, s>>>(P, n_blocks);
    return hipGetLastError();
}

// The dense tables from sorted keys (after a radix sort; the counting sort fills
// them itself).
hipError_t launch_build_dense(const DevParams& P, const uint32_t* skeys, int n, int n_blocks, unsigned* partials,
                              hipStream_t s) {
    const int gb = grid_for(n_blocks);
    k_dense_clear_seg<<<gb, WG, 0, s>>>(P, n_blocks);
    if (n > 0) {
        if (P.dim == 3)
            k_dense_segments<3><<<(n + WG - 1) / WG, WG, 0, s>>>(P, skeys, n);
        else
            k_dense_segments<2><<<(n + WG - 1) / WG, WG, 0, s>>>(P, skeys, n);
    }
    k_dense_counts<<<gb, WG, 0, s>>>(P, n_blocks);
    hipError_t e = scan_exclusive(P.b_chunks, P.b_chunk_off, n_blocks, nullptr, partials,
                                  (unsigned*)&P.ctr->n_work, s);
    if (e != hipSuccess) return e;
    k_work_write<<<gb, WG, 0, s>>>(P);
    return launch_grid_clear(P, n_blocks, s);
}

hipError_t launch_grid_clear(const DevParams& P, int n_blocks, hipStream_t s) {
    const long long NPB = P.dim == 3 ? 64 : 16;
    if (P.dim == 3)
        k_grid_clear<3><<<grid_for((long long)n_blocks * NPB, 65536), WG, 0, s>>>(P, (long long)n_blocks * NPB);
    else
        k_grid_clear<2><<<grid_for((long long)n_blocks * NPB, 65536), WG, 0, s>>>(P, (long long)n_blocks * NPB);
    return hipGetLastError();
}

hipError_t launch_copy_active(const DevParams& P, uint64_t* keys, uint64_t* masks, int cap, hipStream_t s) {
    k_copy_active<<<grid_for(cap, 2048), WG, 0, s>>>(P, keys, masks, cap);
    return hipGetLastError();
}

}  // namespace mpmx
