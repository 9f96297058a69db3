// Incremental re-sort of the particles by owner block: the alternative to the
// full sorts (tabsort.hip, sort.hip) for a build that follows a build of the same
// number of particles on the same context.
//
// The particle at position i of a step's G2P output belongs to the owner
// segment [b_start, b_start + b_count) of the previous build that contains i,
// and a step moves a particle by a fraction of a cell, so nearly all particles
// keep their owner block.  What the later stages need is a grouping, not a
// global order: each owner block's particles contiguous, base cells ascending
// inside the block.  The new layout keeps the previous blocks in their
// previous order and appends the blocks that had no slot before:
//   count    one wave per previous block: the particles whose new key has the
//            block's owner part ("stayers") are counted per base cell and per
//            block (and per RS_TILE blocks), the others ("movers") are listed
//            from the block's first position on (so no list space is claimed
//            from a shared counter), their number with the block's first work
//            item;
//            (inside mpm_step the G2P that wrote the positions does this
//            itself, item by item, see k_g2p)
//   route    one thread per mover, 16 per work item at a time: its new block is looked up in the previous
//            hash table and the block's per-cell mover count and particle
//            count incremented, or, for a block without a previous slot, a
//            slot of a second hash table is claimed (the claiming thread
//            appends it to a list) and counted; the mover's target (entry
//            or slot) is recorded for the placement;
//   place    one wave per entry (the previous blocks, then the listed new ones
//            in claim order).  A previous block's first position is the sum of
//            the particle counts before it: up to FOLD_MAX_N particles each
//            workgroup adds up whole tiles of RS_TILE blocks from their sums
//            and the rest of its own tile count by count, instead of a scan in
//            two launches of its own; a new block's is claimed from a counter
//            past the previous blocks'.  First positions of the entry's cells follow from a
//            wave scan of stayers + movers per cell; for a previous block each
//            stayer then takes the next position of its cell from an LDS
//            counter (an atomic, so stayers of one cell land in any order).
//            The same pass clears the tables the route has finished with: the
//            slots that the previous build occupied and the second table's;
//   finish   two independent jobs in one launch.  One thread per mover: movers
//            go after the stayers of their cell, each taking the position its
//            atomic decrement of the cell's mover count names (which leaves
//            the counts at zero for the next build).  2^d lanes per entry: the
//            entry's block and the blocks its stencils reach go into the block
//            hash (from the base cells that the placement recorded).
// The kernels are short and bound by their dependent memory accesses, so
// launches count: as ten kernels (with compaction and neighbour tables) a
// step's build took 49 us of kernel time at 262,144 particles and 76 us at 2.5 M;
// as these three and the compaction it takes 24 and 45 us.  Per-block kernels only stream keys; the dependent lookups of the
// few movers run one per thread, so their latencies overlap instead of stalling
// a block's wave.
#include <algorithm>

#include "hash.h"

namespace mpmx {

namespace {

// Lanes whose value v (its low BITS bits) equals this lane's, among lanes with
// `valid` set.  Every lane of the wave must call it.
template <int BITS>
__device__ __forceinline__ unsigned long long match_bits(unsigned v, bool valid) {
    unsigned long long m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (v >> b) & 1u;
        const unsigned long long bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// 64-bit block key (Eq. 22, instance folded in) of the owner part of a sort key.
template <int DIM>
__device__ __forceinline__ uint64_t owner_block_key(const DevParams& P, uint32_t owner) {
    const uint32_t bl = owner & ((1u << P.blk_bits) - 1u);
    const int inst = (int)(owner >> P.blk_bits);
    int bc[3];
    linear_to_block<DIM>(P, bl, bc);
    return block_key<DIM>(P, bc[0], bc[1], bc[2], inst);
}

// Second table: same size, hash and probing as the block table.  *claimed is
// set for the one caller whose CAS stored the key.
__device__ int nh_insert(const DevParams& P, uint64_t K, bool* claimed) {
    unsigned s = (unsigned)mix64(K) & P.h_mask_bits;
    *claimed = false;
    for (int r = 0; r < P.n_probe; ++r) {
        const uint64_t cur = __hip_atomic_load(&P.nh_keys[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == K) return (int)s;
        if (cur == EMPTY_KEY) {
            const uint64_t old = atomicCAS((unsigned long long*)&P.nh_keys[s], (unsigned long long)EMPTY_KEY,
                                           (unsigned long long)K);
            *claimed = old == EMPTY_KEY;
            if (old == EMPTY_KEY || old == K) return (int)s;
        }
        s = (s + 1) & P.h_mask_bits;
    }
    return -1;
}

}  // namespace

constexpr int RS_BATCH = 8;  // 64-particle chunks of a segment whose keys are loaded together

// count: one wave per previous block e (its segment of the previous order), and
// the listing of the block's movers.
template <int DIM>
__global__ __launch_bounds__(WG) void k_rs_count(DevParams P, const uint32_t* __restrict__ keys_new,
                                                 uint32_t* __restrict__ movers) {
    constexpr int CB = 2 * DIM, NC = 1 << CB;
    __shared__ unsigned cnt[WG / 64][64];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int nb = min(P.ctr->nb, P.block_cap);
    const int stride = gridDim.x * (WG / 64);
    int s_n = 0, c_n = 0;
    auto fetch = [&](int e) {  // the wave's next block, loaded while the current one is counted
        c_n = 0;
        if (e < nb) {
            asm volatile("" : "+v"(e));  // same in every lane; keeps the values in vector registers
            s_n = P.b_start[e];
            c_n = P.b_count[e];
        }
    };
    fetch(blockIdx.x * (WG / 64) + w);
    for (int e = blockIdx.x * (WG / 64) + w; e < nb; e += stride) {
        const int s = s_n, c = c_n;
        fetch(e + stride);
        cnt[w][lane] = 0u;
        // owner part of the block's sort key, stored by the previous build (a
        // block that only held stencil nodes may still receive movers)
        const uint32_t owner = P.rs_oldblk[e];
        const unsigned items = P.b_chunks[e], it0 = P.b_chunk_off[e];
        unsigned n_mov = 0u;
        if (c > 0) {
            const int end = s + c;
            for (int i0 = s; i0 < end; i0 += 64 * RS_BATCH) {
                uint32_t k[RS_BATCH];
#pragma unroll
                for (int r = 0; r < RS_BATCH; ++r) {
                    const int i = i0 + r * 64 + lane;
                    k[r] = i < end ? keys_new[i] : 0u;
                }
#pragma unroll
                for (int r = 0; r < RS_BATCH; ++r) {
                    if (i0 + r * 64 >= end) break;  // uniform
                    const int i = i0 + r * 64 + lane;
                    const bool valid = i < end;
                    const bool stay = valid && (k[r] >> CB) == owner;
                    const uint32_t cell = k[r] & (NC - 1);
                    const unsigned long long m = match_bits<CB>(cell, stay);
                    if (stay && (m & lt) == 0ull) cnt[w][cell] += (unsigned)__popcll(m);  // one leader per cell
                    const unsigned long long mv = __ballot(valid && !stay);
                    if (valid && !stay) movers[s + n_mov + (unsigned)__popcll(mv & lt)] = (uint32_t)i;
                    n_mov += (unsigned)__popcll(mv);
                }
            }
        }
        if (lane < NC) P.rs_stay[(size_t)e * NC + lane] = cnt[w][lane];
        if (lane == 0) {
            const unsigned tot = (unsigned)max(c, 0) - n_mov;
            P.rs_cnt[e] = tot;
            if (P.rs_tile && tot) atomicAdd(&P.rs_tile[e / RS_TILE * LINE], tot);
        }
        for (unsigned q = lane; q < items; q += 64)
            if (it0 + q < (unsigned)P.work_cap) P.it_mov[it0 + q] = q == 0u ? n_mov : 0u;
    }
}

// route: one thread per mover (16 lanes per work item's list).
// Target of a mover, recorded by the route for the placement: its previous
// entry, or (RS_TGT_NEW | slot) a slot of the second table, or RS_TGT_NONE.
constexpr uint32_t RS_TGT_NEW = 0x80000000u;
constexpr uint32_t RS_TGT_NONE = 0xFFFFFFFFu;

// Calls f(t) for each mover of each work item, t its place in the list; workgroup
// b of nwg workgroups.
template <class F>
__device__ __forceinline__ void for_movers(const DevParams& P, int n, int b, int nwg, F&& f) {
    constexpr int L = 16;  // lanes per list: an item of 512 has a few movers
    const int n_work = min(P.ctr->n_work, P.work_cap);
    const int l = threadIdx.x % L;
    for (int it = (b * WG + (int)threadIdx.x) / L; it < n_work; it += nwg * (WG / L)) {
        const int s = P.w_start[it], c = min((int)P.it_mov[it], n - s);
        for (int j = l; j < c; j += L) f(s + j);
    }
}

template <int DIM>
__global__ __launch_bounds__(WG) void k_rs_route(DevParams P, const uint32_t* __restrict__ keys_new,
                                                 const uint32_t* __restrict__ movers, uint32_t* __restrict__ tgt,
                                                 int n) {
    constexpr int CB = 2 * DIM, NC = 1 << CB;
    for_movers(P, n, blockIdx.x, gridDim.x, [&](int t) {
        const uint32_t k = keys_new[movers[t]];
        const uint32_t cell = k & (NC - 1);
        const uint64_t K = owner_block_key<DIM>(P, k >> CB);
        const int phi = hash_lookup(P, K);
        uint32_t target = RS_TGT_NONE;
        // one add per wave and tile of blocks (the movers of a wave come from a
        // few neighbouring blocks)
        unsigned long long todo = P.rs_tile ? __ballot(phi >= 0) : 0ull;
        while (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const int tile = readlane32(phi, leader) / RS_TILE;
            const unsigned long long same = __ballot(phi >= 0 && phi / RS_TILE == tile);
            if (__lane_id() == leader) atomicAdd(&P.rs_tile[tile * LINE], (unsigned)__popcll(same));
            todo &= ~same;
        }
        if (phi >= 0) {
            atomicAdd(&P.rs_in[(size_t)phi * NC + cell], 1u);
            atomicAdd(&P.rs_cnt[phi], 1u);
            target = (uint32_t)phi;
        } else {
            bool claimed;
            const int slot = nh_insert(P, K, &claimed);
            if (slot >= 0) {
                atomicAdd(&P.nh_cnt[(size_t)slot * NC + cell], 1u);
                P.nh_owner[slot] = k >> CB;  // the same value from every mover of the block
                if (claimed) {
                    // the slot joins the list of new blocks (claim order)
                    const int j = atomicAdd(&P.ctr->rs_n_new, 1);
                    if (j < P.block_cap) P.rs_new[j] = (uint32_t)slot;
                }
                target = RS_TGT_NEW | (uint32_t)slot;
            } else {
                raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
            }
        }
        tgt[t] = target;
    });
}

// Entries of the re-sort: the previous blocks, then the listed new ones.
__device__ __forceinline__ int rs_entries(const DevParams& P, int nb) {
    return min(nb + min(P.ctr->rs_n_new, P.block_cap), 2 * P.block_cap);
}

constexpr int RS_STAGE = 768;  // particles of a block whose output is staged in LDS (larger: direct stores);
                                // 13 KB of LDS per workgroup
constexpr uint32_t RS_EMPTY = 0xFFFFFFFFu;  // staging slot left to a mover (indices are < 2^30)

// place: one wave per entry.  The block's output range (stayers and the movers
// that join it) is staged in LDS and written out contiguously.
// SCANNED: the previous blocks' first positions are in rs_start and their total
// in rs_new_pos (a scan ran before); otherwise each workgroup adds up the counts
// before its four entries, beside the loads of the first.
template <int DIM, bool SCANNED>
__global__ __launch_bounds__(WG) void k_rs_place(DevParams P, const uint32_t* __restrict__ keys_new,
                                                 uint32_t* __restrict__ vals_out, int n, unsigned H) {
    constexpr int CB = 2 * DIM, NC = 1 << CB, NW = WG / 64;
    __shared__ unsigned run[NW][64];
    __shared__ uint32_t sv[NW][RS_STAGE];
    __shared__ unsigned red[NW];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int nb = min(P.ctr->nb, P.block_cap);
    const int n_new = P.ctr->rs_n_new;
    const int ne = rs_entries(P, nb);
    // groups of NW previous blocks, then groups of new ones
    const int gp = (nb + NW - 1) / NW, gn = (ne - nb + NW - 1) / NW;
    // blocks past the list or the entries (reported once)
    bool bad = n_new > ne - nb && blockIdx.x == 0 && threadIdx.x == 0;
    int s_n = 0, c_n = 0;
    unsigned st_n = 0u, in_n = 0u, tot_n = 0u, base_n = 0u;
    uint32_t owner_n = 0u;
    auto fetch = [&](int g) {  // the wave's entry of group g, where that is a previous block
        int e = g * NW + w;
        if (g < gp && e < nb) {
            asm volatile("" : "+v"(e));  // same in every lane; keeps the values in vector registers
            s_n = P.b_start[e];
            c_n = P.b_count[e];
            owner_n = P.rs_oldblk[e];
            tot_n = P.rs_cnt[e];
            if (SCANNED) base_n = P.rs_start[e];
            st_n = lane < NC ? P.rs_stay[(size_t)e * NC + lane] : 0u;
            in_n = lane < NC ? P.rs_in[(size_t)e * NC + lane] : 0u;
        }
    };
    fetch(blockIdx.x);
    for (int g = blockIdx.x; g < gp + gn; g += gridDim.x) {
        const bool prev = g < gp;
        const int e0 = prev ? g * NW : nb + (g - gp) * NW, e = e0 + w;
        const int s = s_n, c = c_n;
        const unsigned st = st_n, in = in_n;
        unsigned tot = tot_n, base = base_n;
        uint32_t owner = owner_n;
        if (!SCANNED) {
            // whole tiles before the group, then the counts of its own tile
            const int tile = prev ? e0 / RS_TILE : (nb + RS_TILE - 1) / RS_TILE;
            const int q = tile * RS_TILE + (int)threadIdx.x;
            static_assert(RS_TILE == WG, "one count per thread");
            unsigned before = prev && q < e0 ? P.rs_cnt[q] : 0u;
            for (int t = threadIdx.x; t < tile; t += WG) before += P.rs_tile[t * LINE];
            const unsigned own = prev && lane < w ? P.rs_cnt[e0 + lane] : 0u;  // the group's entries before the wave's
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
            if (lane == 0) red[w] = before;
            __syncthreads();
            base = 0u;
#pragma unroll
            for (int k = 0; k < NW; ++k) base += red[k] + (unsigned)readlane32((int)own, k);
            __syncthreads();  // red is rewritten in the next round
        }
        fetch(g + gridDim.x);
        if (e >= (prev ? nb : ne)) continue;
        unsigned cv = in;
        if (prev) {
            if (c > 0) cv += st;  // (no row was counted for a block without particles)
        } else {
            const uint32_t slot = P.rs_new[e - nb];
            uint32_t* src = &P.nh_cnt[(size_t)slot * NC];
            owner = P.nh_owner[slot];
            cv = 0u;
            if (lane < NC) {
                cv = src[lane];
                src[lane] = 0u;
                P.rs_in[(size_t)e * NC + lane] = cv;
            }
            if (lane == 0) {
                P.nh_idx[slot] = e;
                P.rs_oldblk[e] = owner;
            }
        }
        const unsigned inc = wave_incl_scan(cv);
        if (!prev) {
            tot = (unsigned)readlane32((int)inc, 63);
            unsigned pos = 0u;
            if (lane == 0) {
                pos = atomicAdd((unsigned*)&P.ctr->rs_new_pos, tot);
                P.rs_cnt[e] = tot;
            }
            base = (SCANNED ? 0u : base) + (unsigned)readlane32((int)pos, 0);
        }
        if (tot == 0u) continue;
        const uint64_t occ = (uint64_t)__ballot(cv != 0u);  // the block's base cells, for the insertion
        const unsigned off = base + inc - cv;
        if (lane == 0) {
            P.rs_start[e] = base;
            P.rs_occ[e] = occ;
        }
        if (lane < NC) {
            P.rs_off[(size_t)e * NC + lane] = off;
            if (prev && c <= 0) P.rs_stay[(size_t)e * NC + lane] = 0u;  // the movers' placement adds it
        }
        if (!prev || c <= 0) continue;
        const bool staged = tot <= (unsigned)RS_STAGE;
        if (staged)
            for (unsigned j = lane; j < tot; j += 64) sv[w][j] = RS_EMPTY;
        run[w][lane] = off;
        const int end = s + c;
        for (int i0 = s; i0 < end; i0 += 64 * RS_BATCH) {
            uint32_t k[RS_BATCH];
#pragma unroll
            for (int r = 0; r < RS_BATCH; ++r) {
                const int i = i0 + r * 64 + lane;
                k[r] = i < end ? keys_new[i] : 0u;
            }
#pragma unroll
            for (int r = 0; r < RS_BATCH; ++r) {
                if (i0 + r * 64 >= end) break;  // uniform
                const int i = i0 + r * 64 + lane;
                const bool stay = i < end && (k[r] >> CB) == owner;
                const uint32_t cell = k[r] & (NC - 1);
                if (stay) {
                    // next position of the cell: an LDS atomic on its counter
                    // (lanes hitting one counter are served one after another,
                    // so any order of them is a valid placement)
                    const unsigned pos = atomicAdd(&run[w][cell], 1u);
                    if (staged && pos - base < tot) {
                        sv[w][pos - base] = (uint32_t)i;
                    } else if (!staged && pos < (unsigned)n) {
                        vals_out[pos] = (uint32_t)i;
                    } else {
                        bad = true;
                    }
                }
            }
        }
        if (staged) {
            for (unsigned j = lane; j < tot; j += 64) {
                const uint32_t v = sv[w][j];
                if (v != RS_EMPTY && base + j < (unsigned)n) vals_out[base + j] = v;
            }
        }
    }
    if (bad) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
    // The tables the route has finished with are cleared here, behind the
    // placement's latency-bound work: of the block hash the slots that the
    // previous build occupied, for the insertion that follows (Algorithm 5's
    // initialisation), and of the second table the listed ones, for the next
    // re-sort.  (The movers' placement reads the route's recorded targets, not
    // the tables.)  Past a capacity the lists are not complete and the whole
    // tables are cleared.
    const int t0 = blockIdx.x * WG + threadIdx.x, tn = gridDim.x * WG;
    const int tiles = ((int)H + SCAN_TILE - 1) / SCAN_TILE;
    for (int t = t0; t < tiles; t += tn) P.t_cnt[t * LINE] = P.t_cnt[t * LINE + 1] = 0u;
    const bool all = P.ctr->n_touched > P.block_cap, all_new = n_new > P.block_cap;
    auto clear = [&](size_t q) {
        P.h_keys[q] = EMPTY_KEY;
        P.h_mask[q] = 0ull;
        P.h_start[q] = -1;
        P.h_end[q] = -1;
        P.h_entry[q] = -1;
    };
    if (all)
        for (long long t = t0; t < (long long)H; t += tn) clear((size_t)t);
    else
        for (int t = t0; t < nb; t += tn) clear((size_t)P.b_hs[t]);
    if (all_new)
        for (long long t = t0; t < (long long)H; t += tn) P.nh_keys[t] = EMPTY_KEY;
    else
        for (int t = t0; t < n_new; t += tn) P.nh_keys[P.rs_new[t]] = EMPTY_KEY;
}

// finish: the first `gm` workgroups place the movers, after the stayers of
// their cells; the others insert the entries' blocks into the block hash, 2^d
// lanes per entry.
template <int DIM>
__global__ __launch_bounds__(WG) void k_rs_finish(DevParams P, const uint32_t* __restrict__ keys_new,
                                                  const uint32_t* __restrict__ movers,
                                                  const uint32_t* __restrict__ tgt, uint32_t* __restrict__ vals_out,
                                                  int n, int gm) {
    constexpr int CB = 2 * DIM, NC = 1 << CB, NB = 1 << DIM;
    const int nb = min(P.ctr->nb, P.block_cap);
    const int ne = rs_entries(P, nb);
    if ((int)blockIdx.x >= gm) {
        // 2^d lanes per entry, one for each block its stencils can reach
        const int lane = __lane_id(), d = lane % NB;
        const int t0 = ((int)blockIdx.x - gm) * WG + (int)threadIdx.x, tn = ((int)gridDim.x - gm) * WG;
        for (int e = t0 / NB; e < ne; e += tn / NB) {
            const unsigned tot = P.rs_cnt[e];
            const unsigned first = P.rs_start[e];
            const uint64_t occ = P.rs_occ[e];
            const uint32_t owner = P.rs_oldblk[e];
            if (tot == 0u) continue;
            const int slot = insert_block<DIM>(P, owner, occ, d);
            const int own = __shfl(slot, lane - d);  // the owner block's
            P.rs_nslot[(size_t)e * NB + d] = slot;
            if (own >= 0 && d == 0) {
                P.h_start[own] = (int)first;
                P.h_end[own] = (int)(first + tot);
                P.h_entry[own] = e;
                atomicAdd(&P.t_cnt[own / SCAN_TILE * LINE + 1], block_chunks(P, (int)tot));
            }
        }
        return;
    }
    bool bad = false;
    for_movers(P, n, blockIdx.x, gm, [&](int t) {
        const uint32_t i = movers[t];
        const uint32_t k = keys_new[i];
        const uint32_t cell = k & (NC - 1);
        const uint32_t target = tgt[t];  // the route's lookup, so no table is probed again
        const bool prev = (target & RS_TGT_NEW) == 0u;
        int e2 = -1;
        if (prev) {
            e2 = (int)target < nb ? (int)target : -1;
        } else if (target != RS_TGT_NONE) {
            e2 = P.nh_idx[target & ~RS_TGT_NEW];
            if (e2 < nb || e2 >= ne) e2 = -1;
        }
        if (e2 < 0) {
            bad = true;
            return;
        }
        const size_t r = (size_t)e2 * NC + cell;
        // the cell's movers still to place, this one included: the last of
        // them takes the first position after the stayers (the decrement and
        // the loads of the cell's offsets are in flight together)
        const unsigned left = atomicSub(&P.rs_in[r], 1u);
        const unsigned b0 = P.rs_off[r] + (prev ? P.rs_stay[r] : 0u);
        const unsigned pos = b0 + left - 1u;
        if (left != 0u && pos < (unsigned)n)
            vals_out[pos] = i;
        else
            bad = true;
    });
    if (bad) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
}

// Initial state of the buffers the re-sort expects between builds.
template <int DIM>
__global__ __launch_bounds__(WG) void k_rs_init(DevParams P, unsigned H) {
    constexpr int NC = 1 << (2 * DIM);
    const long long rows = 2ll * P.block_cap * NC;
    const long long hrows = (long long)H * NC;
    const long long all = rows > hrows ? rows : hrows;
    for (long long t = (long long)blockIdx.x * WG + threadIdx.x; t < all; t += (long long)gridDim.x * WG) {
        if (t < rows) P.rs_in[t] = 0u;
        if (t < hrows) P.nh_cnt[t] = 0u;
        if (t < (long long)H) {
            P.nh_keys[t] = EMPTY_KEY;
            P.nh_idx[t] = -1;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) P.ctr->rs_n_new = 0;
}

namespace {
int grid_for_waves(long long waves) {
    const long long g = (waves + WG / 64 - 1) / (WG / 64);
    return (int)(g < 1 ? 1 : (g > 16384 ? 16384 : g));
}
}  // namespace

hipError_t launch_resort_init(const DevParams& P, unsigned H, hipStream_t s) {
    if (P.dim == 3)
        k_rs_init<3><<<4096, WG, 0, s>>>(P, H);
    else
        k_rs_init<2><<<4096, WG, 0, s>>>(P, H);
    return hipGetLastError();
}

// counted: the G2P that wrote keys_new already stored the stayer counts (per
// previous block and cell, per block, per tile of blocks) and the mover list (in
// any order) with its length; count is skipped.
namespace {
template <int DIM>
hipError_t resort(const DevParams& P, const uint32_t* keys_new, uint32_t* vals_out, uint32_t* movers, uint32_t* tgt,
                  int n, unsigned H, unsigned* partials, hipStream_t s, bool counted) {
    const int ge = grid_for_waves(2ll * P.block_cap);
    const int gi = (int)std::min<long long>((2ll * P.block_cap * (1 << DIM) + WG - 1) / WG, 8192);
    const int gm = std::max(1, std::min((P.work_cap + WG / 16 - 1) / (WG / 16), 2048));
    if (!counted) k_rs_count<DIM><<<grid_for_waves(P.block_cap), WG, 0, s>>>(P, keys_new, movers);
    k_rs_route<DIM><<<gm, WG, 0, s>>>(P, keys_new, movers, tgt, n);
    if (P.rs_tile) {
        k_rs_place<DIM, false><<<ge, WG, 0, s>>>(P, keys_new, vals_out, n, H);
    } else {
        hipError_t e =
            scan_exclusive(P.rs_cnt, P.rs_start, P.block_cap, &P.ctr->nb, partials, (unsigned*)&P.ctr->rs_new_pos, s);
        if (e != hipSuccess) return e;
        k_rs_place<DIM, true><<<ge, WG, 0, s>>>(P, keys_new, vals_out, n, H);
    }
    k_rs_finish<DIM><<<gm + gi, WG, 0, s>>>(P, keys_new, movers, tgt, vals_out, n, gm);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_resort(const DevParams& P, const uint32_t* keys_new, uint32_t* vals_out, uint32_t* movers,
                         uint32_t* tgt, int n, unsigned H, unsigned* partials, hipStream_t s, bool counted) {
    return P.dim == 3 ? resort<3>(P, keys_new, vals_out, movers, tgt, n, H, partials, s, counted)
                      : resort<2>(P, keys_new, vals_out, movers, tgt, n, H, partials, s, counted);
}

}  // namespace mpmx
