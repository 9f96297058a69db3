// Full sort of the particles by (owner block, base cell), stable, by counting in
// a table of every owner block of the potential domain.  Gives exactly the order
// of the radix sort (sort.hip), which serves domains too large for a table
// (TAB_MAX_IDS) and cells too full (TAB_MAX_PER_CELL).
//
//   count    one thread per particle: lanes of a wave that share a block are
//            merged, one add per block and wave claims their places in the
//            block (the order of claims is arbitrary); the hash table is
//            cleared behind it;
//   scan     two launches over the table: first position and entry number of
//            each occupied block, entries in ascending block order;
//   place    one thread per particle: its index goes to its place;
//   order    one workgroup per entry (one wave where blocks are small): the block's indices are counted into its
//            cells and each cell's few indices put in ascending order, which
//            makes the sort stable whatever the claims' order was; permutation
//            and keys are written.  One wave meanwhile inserts the block into
//            the hash table (hash-built grids): its occupied cells are known.
//
// On a dense grid the scan also writes the block tables and work items, as the
// block index is Phi there (it took six launches, 22 us of a step of 262,144 particles
// in 23,465 blocks, less), and P2G walks the entries instead of the domain (30
// us against 40).  For a scan-built context the order leaves each block's
// occupied cells and the counts stay for the build (scanbuild.hip).
//
// The radix sort needs three to four passes of four launches each for these
// keys, all bound by latency at moderate sizes; with the hash clearing, the
// insertion (which served a wave's blocks one after another) and the item
// count a full build took 16-21 launches before the compaction.  Here each of
// the five is a short chain of dependent accesses: at 262,144 particles in order
// 4.8 us for the count, 3.9 and 4.5 for the scan, 2.8 for the places, 9.4 for the
// order with the insertion, where three radix passes took 69, the insertion 20
// and clearing and item count 9.  (A wave per block that ordered each cell by
// insertion and only then inserted its block took 16.)
#include <algorithm>
#include <climits>

#include "hash.h"

namespace mpmx {

namespace {

// Per tile of WG ITEMS table entries: particles and occupied blocks; DENSE: work
// items; SCAN: bounding box of the occupied blocks.
template <int DIM, TabMode MODE, int ITEMS>
__global__ __launch_bounds__(WG) void k_tab_reduce(DevParams P, TabSort T) {
    __shared__ unsigned lds[WG / 64];
    __shared__ int red[WG / 64][6];
    const int base = blockIdx.x * (WG * ITEMS) + threadIdx.x;
    unsigned c = 0, z = 0, w = 0, v[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) v[j] = base + j * WG < T.ids ? T.cnt[base + j * WG] : 0u;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        c += v[j];
        z += v[j] != 0u ? 1u : 0u;
        if (MODE == TAB_DENSE) w += block_chunks(P, (int)v[j]);
    }
    unsigned tc, tz, tw = 0u;
    wg_excl_scan(c, lds, &tc);
    wg_excl_scan(z, lds, &tz);
    if (MODE == TAB_DENSE) wg_excl_scan(w, lds, &tw);
    if (threadIdx.x == 0) {
        T.part[4 * blockIdx.x] = tc;
        T.part[4 * blockIdx.x + 1] = tz;
        T.part[4 * blockIdx.x + 2] = tw;
    }
    if (MODE == TAB_SCAN) {
        int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {-1, -1, -1};
        if (tz != 0u) {
#pragma unroll 1
            for (int j = 0; j < ITEMS; ++j) {
                if (base + j * WG >= T.ids || T.cnt[base + j * WG] == 0u) continue;
                int bc[3];
                linear_to_block<DIM>(P, (uint32_t)(base + j * WG), bc);
#pragma unroll
                for (int a = 0; a < DIM; ++a) {
                    lo[a] = min(lo[a], bc[a]);
                    hi[a] = max(hi[a], bc[a]);
                }
            }
        }
        box_reduce(lo, hi, red);
        if (threadIdx.x == 0)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T.box[8 * blockIdx.x + a] = lo[a];
                T.box[8 * blockIdx.x + 4 + a] = hi[a];
            }
    }
}

template <TabMode MODE, int ITEMS>
__global__ __launch_bounds__(WG) void k_tab_down(DevParams P, TabSort T, int tiles) {
    __shared__ unsigned lds[WG / 64], red[WG / 64][5];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int base = blockIdx.x * (WG * ITEMS) + threadIdx.x * ITEMS;
    unsigned v[ITEMS], s[5] = {0u, 0u, 0u, 0u, 0u}, c = 0u, z = 0u, it = 0u;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) v[j] = base + j < T.ids ? T.cnt[base + j] : 0u;
    // sums of the tiles before this one, and the occupied blocks (DENSE: and
    // the work items) of all
    for (int i = threadIdx.x; i < tiles; i += WG) {
        const uint4 p = *(const uint4*)&T.part[4 * i];
        const bool before = i < (int)blockIdx.x;
        s[0] += before ? p.x : 0u;
        s[1] += before ? p.y : 0u;
        s[2] += p.y;
        if (MODE == TAB_DENSE) {
            s[3] += before ? p.z : 0u;
            s[4] += p.z;
        }
    }
    constexpr int NS = MODE == TAB_DENSE ? 5 : 3;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int q = 0; q < NS; ++q) s[q] += __shfl_xor(s[q], o);
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < NS; ++q) red[w][q] = s[q];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        c += v[j];
        z += v[j] != 0u ? 1u : 0u;
        if (MODE == TAB_DENSE) it += block_chunks(P, (int)v[j]);
    }
    unsigned tot;
    unsigned pos = wg_excl_scan(c, lds, &tot);
    unsigned ent = wg_excl_scan(z, lds, &tot);  // its barriers also publish red
    unsigned item = MODE == TAB_DENSE ? wg_excl_scan(it, lds, &tot) : 0u;
    unsigned all = 0u, items = 0u;
#pragma unroll
    for (int q = 0; q < WG / 64; ++q) {
        pos += red[q][0];
        ent += red[q][1];
        all += red[q][2];
        if (MODE == TAB_DENSE) {
            item += red[q][3];
            items += red[q][4];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *T.n_ent = (int)all;
        if (MODE == TAB_DENSE) {
            P.ctr->nb = T.ids;
            P.ctr->n_touched = T.ids;
            P.ctr->n_work = (int)items;
        }
    }
    bool over = false;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int b = base + j;
        if (MODE == TAB_DENSE && b < T.ids) {
            const unsigned k = block_chunks(P, (int)v[j]);
            P.b_start[b] = v[j] != 0u ? (int)pos : -1;
            P.b_count[b] = (int)v[j];
            P.b_chunks[b] = k;
            for (unsigned q = 0; q < k; ++q) {
                if (item + q >= (unsigned)P.work_cap) {
                    over = true;
                    break;
                }
                P.w_block[item + q] = b;
                P.w_start[item + q] = (int)pos + (int)q * P.chunk;
                P.w_end[item + q] = (int)(pos + min((q + 1u) * (unsigned)P.chunk, v[j]));
            }
            item += k;
        }
        if (v[j] == 0u) continue;
        T.start[b] = pos;
        if (MODE == TAB_SCAN) T.eidx[b] = (int)ent;
        if ((int)ent < T.ent_cap) T.ent[ent] = make_uint4((unsigned)b, pos, v[j], 0u);
        pos += v[j];
        ++ent;
    }
    if (over) raise_flag(P.ctr, MPM_FLAG_OVERFLOW);
}

}  // namespace

template <int DIM, bool HASH>
__global__ __launch_bounds__(WG) void k_tab_count(DevParams P, TabSort T, const uint32_t* __restrict__ keys,
                                                  uint32_t* __restrict__ rank, int n, unsigned H) {
    constexpr int CB = 2 * DIM, NB = 1 << DIM;
    const int i = blockIdx.x * WG + threadIdx.x, lane = __lane_id();
    const bool valid = i < n;
    const uint32_t id = valid ? min(keys[i] >> CB, (uint32_t)T.ids - 1u) : ~0u;
    // lanes of the same block: the first of them claims places for all
    unsigned long long todo = __ballot(valid), grp = 0ull;
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const unsigned long long same = __ballot(valid && id == (uint32_t)readlane32((int)id, leader));
        if ((same >> lane) & 1ull) grp = same;
        todo &= ~same;
    }
    const int leader = grp ? __ffsll((long long)grp) - 1 : lane;
    unsigned first = 0u;
    if (valid && lane == leader) first = atomicAdd(&T.cnt[id], (unsigned)__popcll(grp));
    first = (unsigned)__shfl((int)first, leader);
    if (valid) rank[i] = first + (unsigned)__popcll(grp & ((1ull << lane) - 1ull));
    if (HASH) clear_hash<NB, false>(P, H, blockIdx.x * WG + threadIdx.x, gridDim.x * WG);
}

template <int CB>
__global__ __launch_bounds__(WG) void k_tab_place(TabSort T, const uint32_t* __restrict__ keys,
                                                  const uint32_t* __restrict__ rank, uint32_t* __restrict__ tmp, int n) {
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i >= n) return;
    const unsigned pos = T.start[min(keys[i] >> CB, (uint32_t)T.ids - 1u)] + rank[i];
    if (pos < (unsigned)n) tmp[pos] = (uint32_t)i;
}

namespace {

// A block too full for LDS: LSD radix passes by the wave over its c indices
// (8-bit digits of the index, then the cell), a -> b -> a ..., ending in b.
// cnt64: particles per cell on return (lane = cell).
template <int CB>
__device__ void wave_radix(uint32_t* a, uint32_t* b, int c, int idx_bits, const uint32_t* __restrict__ keys,
                           unsigned* hist, int lane, unsigned* cnt64) {
    constexpr int NC = 1 << CB;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int passes = (idx_bits + 7) / 8 + 1;
    auto ld = [](uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    uint32_t* const out = b;
    for (int p = 0; p < passes; ++p) {
        const bool cells = p == passes - 1;
        auto digit = [&](uint32_t v) { return cells ? keys[v] & (NC - 1) : (v >> (8 * p)) & 255u; };
        for (int q = lane; q < 256; q += 64) hist[q] = 0u;
        for (int i = lane; i < c; i += 64) atomicAdd(&hist[digit(ld(a + i))], 1u);
        if (cells) *cnt64 = lane < NC ? hist[lane] : 0u;
        unsigned h[4], s = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            h[q] = hist[4 * lane + q];
            s += h[q];
        }
        unsigned e = wave_incl_scan(s) - s;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            hist[4 * lane + q] = e;
            e += h[q];
        }
        for (int i0 = 0; i0 < c; i0 += 64) {
            const bool valid = i0 + lane < c;
            const uint32_t v = valid ? ld(a + i0 + lane) : 0u;
            const unsigned d = valid ? digit(v) : 0u;
            unsigned long long m = __ballot(valid);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const bool bit = (d >> q) & 1u;
                const unsigned long long bb = __ballot(bit);
                m &= bit ? bb : ~bb;
            }
            const unsigned at = hist[d];
            if (valid) {
                b[at + (unsigned)__popcll(m & lt)] = v;
                if ((m & lt) == 0ull) hist[d] = at + (unsigned)__popcll(m);
            }
        }
        __threadfence();
        uint32_t* t = a;
        a = b;
        b = t;
    }
    if (a != out) {  // an even number of passes ended in the source
        for (int i = lane; i < c; i += 64) out[i] = ld(a + i);
        __threadfence();
    }
}

}  // namespace

namespace {

// What the rest of the build reads of entry e, each by one wave (m, f: particles and
// first place of cell `lane`, for lanes below 4^d): the cell ranges, beside the
// emptied table ...
template <int DIM, TabMode MODE>
__device__ __forceinline__ void tab_entry_row(const DevParams& P, const TabSort& T, int e, uint32_t id, int st,
                                              unsigned f, int lane) {
    constexpr int NC = 1 << (2 * DIM);
    if (e < P.row_cap && lane < NC) P.rs_off[(size_t)e * NC + lane] = (unsigned)st + f;
    if (MODE != TAB_SCAN && lane == 0) T.cnt[id] = 0u;  // the table is left empty (a scan build empties it itself)
}
// ... the block's cells and its insertion into the hash.
template <int DIM, TabMode MODE>
__device__ __forceinline__ void tab_entry_insert(const DevParams& P, const TabSort& T, int e, uint32_t id, int st,
                                                 int c, unsigned m, int lane) {
    constexpr int NC = 1 << (2 * DIM), NB = 1 << DIM;
    if (MODE == TAB_DENSE) return;
    const uint64_t occ = (uint64_t)__ballot(lane < NC && m != 0u);
    if (MODE == TAB_SCAN && lane == 0) T.occ[id] = occ;
    if (MODE != TAB_HASH) return;
    const int slot = lane < NB ? insert_block<DIM>(P, id, occ, lane) : -1;
    const int own = readlane32(slot, 0);
    if (own < 0) return;
    const bool row = e < P.row_cap;  // with the cell ranges, for P2G
    if (lane < NB) {
        if (row)
            P.rs_nslot[(size_t)e * NB + lane] = slot;
        else
            P.h_nslot[(size_t)own * NB + lane] = slot;
    }
    if (lane == 0) {
        P.h_start[own] = st;
        P.h_end[own] = st + c;
        if (row) P.h_entry[own] = e;
        atomicAdd(&P.t_cnt[own / SCAN_TILE * LINE + 1], block_chunks(P, c));
    }
}

// The order of a block of at most TAB_WAVE particles, by one wave (sidx, scell, cnt,
// first: its own).
template <int DIM, TabMode MODE>
__device__ __forceinline__ void tab_order_wave(const DevParams& P, const TabSort& T, int e, uint4 en, int n,
                                               const uint32_t* __restrict__ keys, const uint32_t* tmp, uint32_t* order,
                                               uint32_t* skeys, uint32_t* sidx, unsigned char* scell, unsigned* cnt,
                                               unsigned* first, int lane) {
    constexpr int CB = 2 * DIM, NC = 1 << CB, R = TAB_WAVE / 64;
    const uint32_t id = en.x;
    const int st = (int)en.y, c = min((int)en.z, n - st);
    auto fence = [] {  // a wave's LDS accesses are served in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    uint32_t ix[R];
    unsigned cl[R], at[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ix[r] = r * 64 + lane < c ? tmp[st + r * 64 + lane] : 0u;
    if (lane < NC) cnt[lane] = 0u;
    fence();
#pragma unroll
    for (int r = 0; r < R; ++r) cl[r] = r * 64 + lane < c ? keys[ix[r]] & (NC - 1) : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) at[r] = r * 64 + lane < c ? atomicAdd(&cnt[cl[r]], 1u) : 0u;
    fence();
    const unsigned m = lane < NC ? cnt[lane] : 0u, f = wave_incl_scan(m) - m;
    if (lane < NC) first[lane] = f;
    fence();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * 64 + lane < c) {
            const unsigned p = first[cl[r]] + at[r];
            sidx[p] = ix[r];
            scell[p] = (unsigned char)cl[r];
        }
    fence();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = r * 64 + lane;
        if (j >= c) continue;
        const uint32_t v = sidx[j];
        const unsigned k = scell[j], f0 = first[k], mk = cnt[k];
        unsigned to = f0;
        for (unsigned q = 0; q < mk; ++q) to += sidx[f0 + q] < v ? 1u : 0u;
        order[st + to] = v;
        skeys[st + to] = (id << CB) | k;
    }
    tab_entry_row<DIM, MODE>(P, T, e, id, st, f, lane);
    tab_entry_insert<DIM, MODE>(P, T, e, id, st, c, m, lane);
    fence();  // (the next entry writes the same LDS)
}

}  // namespace

// tmp and skeys may be one buffer: a block's range is read before it is written.
// One workgroup per occupied block, or (WAVES, where cells at rest put TAB_WAVE_MEAN
// particles or fewer in a block) one wave per block that fits it (a block's chain of
// dependent accesses is as long for 16 particles as for 500, so what counts is how
// many blocks are in flight: 63,504 2D blocks of 63 in 93 us, by a workgroup each in
// 208; 251,990 of 16 in 368 and 885).
// A workgroup's block: its particles are listed cell by cell in
// LDS, then each counts the smaller indices of its cell: no step depends on the
// one before it, where ordering a cell by insertion is a chain of LDS accesses.
template <int DIM, TabMode MODE, bool WAVES>
__global__ __launch_bounds__(WG) void k_tab_order(DevParams P, TabSort T, const uint32_t* __restrict__ keys,
                                                  uint32_t* tmp, uint32_t* order, uint32_t* skeys, int n, int idx_bits) {
    constexpr int CB = 2 * DIM, NC = 1 << CB, R = TAB_BATCH / WG;
    extern __shared__ uint32_t sidx[];                              // T.stage indices
    unsigned char* const scell = (unsigned char*)(sidx + T.stage);  // and their cells
    __shared__ unsigned cnt[NC], first[NC], hist[256];
    const int lane = __lane_id(), t = threadIdx.x;
    const int ne = min(*T.n_ent, T.ent_cap);
    // entries of a workgroup at a time: GS in a row, then GS past the other workgroups'
    constexpr int GS = WAVES ? WG / 64 : 1;
    for (int e = blockIdx.x * GS; e < ne; e += e % GS == GS - 1 ? (gridDim.x - 1) * GS + 1 : 1) {
        if (WAVES) {
            if (e % GS == 0) {  // every wave its own
                const int w = t >> 6, ew = e + w;
                constexpr int WAVE_LDS = TAB_WAVE * 4 + 2 * NC * 4 + TAB_WAVE;
                static_assert(WG / 64 * WAVE_LDS <= TAB_STAGE * 5, "the waves share the staging");
                uint32_t* const wi = (uint32_t*)((char*)sidx + w * WAVE_LDS);
                const uint4 we = ew < ne ? T.ent[ew] : make_uint4(0u, 0u, ~0u, 0u);
                if (we.z <= (unsigned)TAB_WAVE)
                    tab_order_wave<DIM, MODE>(P, T, ew, we, n, keys, tmp, order, skeys, wi,
                                              (unsigned char*)(wi + TAB_WAVE + 2 * NC), wi + TAB_WAVE,
                                              wi + TAB_WAVE + NC, lane);
            }
            if (T.ent[e].z <= (unsigned)TAB_WAVE) continue;
            __syncthreads();  // the waves have finished with the staging
        }
        const uint4 en = T.ent[e];
        const uint32_t id = en.x;
        const int st = (int)en.y, c = min((int)en.z, n - st);
        const bool staged = c <= T.stage;
        if (t < NC) cnt[t] = 0u;
        __syncthreads();
        if (staged && c > TAB_BATCH) {
            // more particles than the registers hold: counted, then read again
            auto batch = [&](auto&& f) {
                for (int r0 = 0; r0 < c; r0 += R * WG) {
                    uint32_t ix[R];
                    unsigned cl[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) ix[r] = r0 + r * WG + t < c ? tmp[st + r0 + r * WG + t] : 0u;
#pragma unroll
                    for (int r = 0; r < R; ++r) cl[r] = r0 + r * WG + t < c ? keys[ix[r]] & (NC - 1) : 0u;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (r0 + r * WG + t < c) f(ix[r], cl[r]);
                }
            };
            batch([&](uint32_t, unsigned cl) { atomicAdd(&cnt[cl], 1u); });
            __syncthreads();
            if (t < 64) {
                const unsigned m = t < NC ? cnt[t] : 0u, f = wave_incl_scan(m) - m;
                if (t < NC) first[t] = hist[t] = f;
            }
            __syncthreads();
            batch([&](uint32_t ix, unsigned cl) {
                const unsigned p = atomicAdd(&hist[cl], 1u);
                sidx[p] = ix;
                scell[p] = (unsigned char)cl;
            });
        } else if (staged) {
            uint32_t ix[R];
            unsigned cl[R], at[R];
#pragma unroll
            for (int r = 0; r < R; ++r) ix[r] = r * WG + t < c ? tmp[st + r * WG + t] : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r) cl[r] = r * WG + t < c ? keys[ix[r]] & (NC - 1) : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r * WG + t < c) at[r] = atomicAdd(&cnt[cl[r]], 1u);
            __syncthreads();
            if (t < 64) {
                const unsigned m = t < NC ? cnt[t] : 0u, f = wave_incl_scan(m) - m;
                if (t < NC) first[t] = f;
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r * WG + t < c) {
                    const unsigned p = first[cl[r]] + at[r];
                    sidx[p] = ix[r];
                    scell[p] = (unsigned char)cl[r];
                }
        } else if (t < 64) {
            unsigned m = 0u;
            wave_radix<CB>(tmp + st, order + st, c, idx_bits, keys, hist, lane, &m);
            const unsigned f = wave_incl_scan(m) - m;
            if (t < NC) {
                cnt[t] = m;
                first[t] = f;
            }
        }
        __syncthreads();
        if (t < 64) tab_entry_row<DIM, MODE>(P, T, e, id, st, t < NC ? first[t] : 0u, t);
        if (t >= WG - 64)  // (the wave with the fewest particles)
            tab_entry_insert<DIM, MODE>(P, T, e, id, st, c, lane < NC ? cnt[lane] : 0u, lane);
        if (staged) {
            for (int j = t; j < c; j += WG) {
                const uint32_t v = sidx[j];
                const unsigned cl = scell[j], f = first[cl], m = cnt[cl];
                unsigned at = f;
                for (unsigned q = 0; q < m; ++q) at += sidx[f + q] < v ? 1u : 0u;
                order[st + at] = v;
                skeys[st + at] = (id << CB) | cl;
            }
        } else {
            for (int j = t; j < c; j += WG)
                skeys[st + j] = (id << CB) |
                                (keys[__hip_atomic_load(order + st + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] &
                                 (NC - 1));
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(WG) void k_tab_init(TabSort T) {
    for (int t = blockIdx.x * WG + threadIdx.x; t < T.ids; t += gridDim.x * WG) {
        T.cnt[t] = 0u;
        if (T.occ) T.occ[t] = 0ull;
    }
}

hipError_t launch_tab_init(const TabSort& T, hipStream_t s) {
    k_tab_init<<<std::max(1, std::min((T.ids + WG - 1) / WG, 2048)), WG, 0, s>>>(T);
    return hipGetLastError();
}

namespace {
template <int DIM, TabMode MODE>
hipError_t tab_sort(const DevParams& P, const TabSort& T, const uint32_t* keys, uint32_t* rank, uint32_t* tmp,
                    uint32_t* order, uint32_t* skeys, int n, unsigned H, hipStream_t s) {
    constexpr bool HASH = MODE == TAB_HASH;
    const int items = tab_items(T.ids, MODE == TAB_SCAN);
    const int g = (n + WG - 1) / WG, tiles = (T.ids + WG * items - 1) / (WG * items);
    const int go = std::max(1, std::min(T.ent_cap, 2048));  // what the chip holds
    int bits = 1;
    while (bits < 30 && (1 << bits) < n) ++bits;
    // (hash: at least 64 workgroups for the clearing)
    if (n > 0) k_tab_count<DIM, HASH><<<HASH ? std::max(g, 64) : g, WG, 0, s>>>(P, T, keys, rank, n, H);
    if (MODE != TAB_SCAN && items == TAB_SMALL_ITEMS) {
        k_tab_reduce<DIM, MODE, TAB_SMALL_ITEMS><<<tiles, WG, 0, s>>>(P, T);
        k_tab_down<MODE, TAB_SMALL_ITEMS><<<tiles, WG, 0, s>>>(P, T, tiles);
    } else {
        k_tab_reduce<DIM, MODE, SCAN_ITEMS><<<tiles, WG, 0, s>>>(P, T);
        k_tab_down<MODE, SCAN_ITEMS><<<tiles, WG, 0, s>>>(P, T, tiles);
    }
    if (n > 0) {
        k_tab_place<2 * DIM><<<g, WG, 0, s>>>(T, keys, rank, tmp, n);
        const auto k = T.waves ? k_tab_order<DIM, MODE, true> : k_tab_order<DIM, MODE, false>;
        k<<<go, WG, (size_t)T.stage * 5, s>>>(P, T, keys, tmp, order, skeys, n, bits);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_tab_sort(const DevParams& P, const TabSort& T, const uint32_t* keys, uint32_t* rank, uint32_t* tmp,
                           uint32_t* order, uint32_t* skeys, int n, unsigned H, TabMode mode, hipStream_t s) {
    const bool d3 = P.dim == 3;
    const auto f = mode == TAB_HASH    ? (d3 ? tab_sort<3, TAB_HASH> : tab_sort<2, TAB_HASH>)
                   : mode == TAB_DENSE ? (d3 ? tab_sort<3, TAB_DENSE> : tab_sort<2, TAB_DENSE>)
                                       : (d3 ? tab_sort<3, TAB_SCAN> : tab_sort<2, TAB_SCAN>);
    return f(P, T, keys, rank, tmp, order, skeys, n, H, s);
}

}  // namespace mpmx
