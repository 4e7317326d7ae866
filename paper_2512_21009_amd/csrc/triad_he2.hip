// triad_he2.hip -- hyperedge-family triad deltas without 2-hop expansion.
//
// Every live hyperedge x carries a histogram H_x over its line-graph
// neighbours y: H_x[k][f] = #{y : |x & y| = k, [|y| > k] = f} (2|x| u32
// counters, stored beside its h2v block).  A changed hyperedge adds or removes
// one neighbour of each x in N(h), so the histograms are kept exact with one
// atomic per (h, x) pair.
//
// For a centre h and a neighbour x, the triads {h, x, y} with y outside the
// closed neighbourhood of h (open paths h - x - y) have the class
//   h only  = |h| > c_x,  x only = |x| - c_x - |x & y| > 0,  y only = |y| > |x & y|,
//   plus the regions h&x and x&y,
// so they are counted from H_x with one threshold (|x & y| < |x| - c_x), minus
// h itself, minus the batch members that rank below h (read from x's
// batch-neighbour list) and, in the pair phase, minus the other neighbours of h
// that meet x.
// Neighbour pairs {x, y} of h that intersect get their true class in place of the
// disjoint-pair class that the histogram pass gave them.  Those that meet inside h are
// counted by kind: neighbours with the same mask of shared members (and the same few other
// bits) change the classes alike, so the pairs are taken between a few dozen kinds.  Those
// that meet outside h are found along the runs of the vertices that two or more neighbours
// share: a wave takes a neighbour x, walks the runs of x's shared vertices and counts them
// for every later neighbour y in LDS counters indexed by the neighbour's number (no hash, no
// sort), then takes each y whose counter is not zero.  A hyperedge of more members than a
// mask holds finds all its pairs along the runs.
//
// What bounds it: gathers (lists, metas, rows, histograms: about six lines of 128 B per
// neighbour) and the latency of their chains, so rows, histograms and lists are walked end
// to end, four steps' loads in flight, with as many waves as the LDS holds.  Measured with
// 100k changes on 2M hyperedges of up to 64 members (both phases): sorted entries and pairs
// enumerated per shared vertex 37.5 ms; counters along all runs 34.8; kinds and flat walks
// 13.7; now 13.0.  5k changes on 500k hyperedges, where two dense centres went to the 2-hop kernel:
// 134 ms, 9.7, 3.0.
#include <type_traits>

#include "triad_common.h"

namespace {

using namespace tri;

// Stage 0: 24 KB of LDS tables, 256 threads, four workgroups per CU.  Stage 1: 54 KB, 512
// threads, two workgroups per CU (one of 1024 threads and 118 KB: 6.6 ms against 3.5 for the
// centres of 100k changes on 2M hyperedges that stage 0 moves on), unless the launch has at
// most two centres per CU: then that one large workgroup, which has the CU to itself anyhow
// and keeps denser centres out of global memory.  Whole batches, two workgroups against one
// large one: n + n changes among 1,000 hub-heavy hyperedges 2.85 -> 1.79 ms at n = 100 and 5.73
// -> 3.43 at 500; one change among 20,000, stages 1 and 2, 0.21 -> 0.15; temporal centres 0.97 ->
// 0.77 ms at n = 64, 2.11 -> 2.07 at 500.  It loses where the centres outgrow 118 KB too (n = 500
// among 3,000 of those hyperedges 25.1 against 25.8 ms, n = 130 among 1,520 5.64 against 6.52)
// and gains less as the launch grows: among 500k hyperedges n = 400 2.259 against 2.266, 512
// 1.924 against 1.968, and beyond the line 800 2.730 against 2.760; 2,000 on 36,000 5.43 against
// 5.72.  Stage 2 (the global stage): tables in global memory, 512 threads, two workgroups per CU.
constexpr uint32_t ARENA_S = 6144;
constexpr uint32_t ARENA_M = 13824;
constexpr uint32_t ARENA_W = 30208;
constexpr int WG_M = 512, WG_L = 512, WG_W = 1024;
constexpr uint32_t CNT_L = 1536;       // stage 2: counter words per wave
constexpr uint32_t LDS_L = 12800;      // ... LDS words: counters of 8 waves, or bitmaps, or a (c, f) histogram
static_assert(LDS_L >= (WG_L / 64) * CNT_L, "global stage LDS");
constexpr uint32_t MASK_BITS = 64;     // hyperedges of up to this many members: a neighbour's shared
                                       // members are one 64-bit mask
constexpr uint32_t K_MAX_N = 1u << 24; // neighbours of a centre (a run cursor and its flag share a word)

// open-addressing tables of any capacity: slot = multiply-shift hash scaled to cap
__device__ __forceinline__ uint32_t fr_slot(uint32_t key, uint32_t cap) {
    return (uint32_t)(((uint64_t)(key * 2654435761u) * cap) >> 32);
}
__device__ __forceinline__ uint32_t fr_next(uint32_t s, uint32_t cap) { return s + 1 == cap ? 0 : s + 1; }
__device__ __forceinline__ uint32_t hash_cap(uint32_t n) { return n + n / 2 + 32; }  // load <= 2/3

// Adds inc to key's value and returns key's slot.
__device__ __forceinline__ uint32_t fr_add(uint32_t* keys, uint32_t* vals, uint32_t cap, uint32_t key, uint32_t inc) {
    uint32_t s = fr_slot(key, cap);
    for (uint32_t probe = 0; probe < cap; probe++) {
        uint32_t k = __atomic_load_n(&keys[s], __ATOMIC_RELAXED);
        if (k == HGT_EMPTY) {
            uint32_t prev = atomicCAS(&keys[s], HGT_EMPTY, key);
            if (prev == HGT_EMPTY || prev == key) { atomicAdd(&vals[s], inc); return s; }
        } else if (k == key) {
            atomicAdd(&vals[s], inc);
            return s;
        }
        s = fr_next(s, cap);
    }
    return 0;  // unreachable: tables hold more slots than keys
}

// A word that atomics write: in global memory they act in the L2, so it is read there.
template <bool GLOBAL>
__device__ __forceinline__ uint32_t ld_at(const uint32_t* p) {
    if (GLOBAL) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}

// What the kernels below call is inlined throughout: one call that takes the parameter
// block by reference puts a copy of the block in scratch, and every field is then read from
// there (the global stage: 5.85 -> 5.61 ms for 100k changes on 2M hyperedges).
struct Sh2 {
    uint32_t h, rank, hlen, lh, K, W, S, defer, stop, rows;
    uint32_t gi, cur_g, skip;
    uint32_t slice, nslice;
    uint64_t hoff;
    uint32_t ws[WG_W / 64];
    uint32_t G;
    uint64_t g[8];
};

// ---- per-centre neighbourhood (shared by the neighbour pass and the delta kernel)
// Builds N(h) -> c_x in the hash at keys/vals (already cleared), reading the
// incidence lists of h's members through pre/voff.
__device__ __forceinline__ void build_nh(const GraphView& G, uint32_t h, uint32_t hlen, uint32_t lh, const uint32_t* pre,
                                         const uint64_t* voff, uint32_t* keys, uint32_t* vals, uint32_t cap,
                                         bool in_window, int64_t window) {
    const int64_t lo = in_window ? ts_sub(G.h_ts[h], window) : 0, hi = in_window ? ts_add(G.h_ts[h], window) : 0;
    for (uint32_t p = threadIdx.x; p < lh; p += HGT_WG) {
        uint32_t k = seg_of<uint32_t>(pre, hlen, p);
        const uint64_t at = voff[k] + (p - pre[k]);
        uint32_t x = G.v2h[at];
        if (in_window) {
            const int64_t t = G.v2h_ts[at];
            if (t < lo || t > hi) continue;
        }
        if (x != h) (void)fr_add(keys, vals, cap, x, 1u);
    }
}

// prefix of member degrees and their list offsets; returns lh (all threads)
__device__ __forceinline__ uint32_t member_prefix(const GraphView& G, uint64_t hoff, uint32_t hlen, uint32_t* pre,
                                                  uint64_t* voff, uint32_t* ws) {
    uint32_t carry = 0;
    for (uint32_t b = 0; b < hlen; b += HGT_WG) {
        uint32_t i = b + threadIdx.x, d = 0;
        if (i < hlen) {
            uint32_t m = G.h2v[hoff + i];
            d = G.v_len[m];
            voff[i] = G.v_off[m];
        }
        uint32_t tot;
        uint32_t ex = wg_scan_u32(d, ws, &tot);
        if (i < hlen) pre[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) pre[hlen] = carry;
    __syncthreads();
    return carry;
}

// ===========================================================================
// neighbour pass: batch-neighbour entries (x, d, k = |x & d|, [|d| > k]) and,
// for inserted hyperedges, the histogram updates
// ===========================================================================
// Words a centre's tables take in the arena: hash, member prefix and offsets.
__device__ __forceinline__ uint64_t nbr_words(uint32_t hlen, uint32_t lh) {
    return 2ull * hash_cap(lh) + 3ull * hlen + 4;
}

constexpr uint32_t NBR_TAKE = 8;  // centres a workgroup takes at once

template <bool BIG>
__device__ __forceinline__ void nbr_pass_body(const NbrParams& P, uint32_t* arena, uint64_t arena_words) {
    __shared__ Sh2 sh;
    __shared__ uint32_t c_gi[NBR_TAKE], c_h[NBR_TAKE], c_rank[NBR_TAKE], c_lh[NBR_TAKE];
    __shared__ uint64_t c_off[NBR_TAKE];
    // An inserted hyperedge's own histogram, as far as it goes here: nearly all neighbours share
    // one or two members with it, so their additions meet at a few words (50k inserts and 50k
    // deletions on 2M hyperedges, additions in global memory: 1.74 ms for both, here 1.09).
    constexpr uint32_t OWN = 128;
    __shared__ uint32_t own[OWN];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t n = BIG ? (uint64_t)*P.big_count : P.M.total;
    uint32_t take = BIG ? 1 : take_size(n, gridDim.x, 4);
    if (take > NBR_TAKE) take = NBR_TAKE;
    for (;;) {
        if (tid == 0) {
            const uint32_t q = atomicAdd(BIG ? P.big_queue : P.queue, take);
            sh.stop = q >= n;
            sh.h = q;                                              // the first of
            sh.K = sh.stop ? 0 : (uint32_t)(n - q < take ? n - q : take);  // this many centres
        }
        __syncthreads();
        if (sh.stop) break;
        const uint32_t q0 = sh.h, nc = sh.K;
        // their member lists' lengths: they bound the entries, so the centres' ranges of
        // the entry array are reserved with one atomic
        for (uint32_t ci = wave; ci < nc; ci += NWAVE) {
            uint32_t gi, h, rank;
            if (BIG) {
                const uint64_t it = P.big_list[q0 + ci];
                gi = (uint32_t)(it >> 32);
                h = (uint32_t)it;
                rank = P.big_rank[q0 + ci];
            } else {
                gi = multi_graph_of(P.M, q0 + ci);
                rank = (uint32_t)(q0 + ci - P.M.base[gi]);
                h = P.M.graphs[gi].centres[rank];
            }
            const HeGraph& Gq = P.M.graphs[gi];
            const bool skip = *((volatile const int32_t*)Gq.status) != 0;
            const uint32_t hlen = skip ? 0 : Gq.g.h_len[h];
            uint32_t lh = 0;
            if (hlen) {
                const uint32_t* row = Gq.g.h2v + Gq.g.h_off[h];
                for (uint32_t i = lane; i < hlen; i += 64) lh += Gq.g.v_len[row[i]];
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) lh += __shfl_xor(lh, o, 64);
            if (lane == 0) {
                c_gi[ci] = gi;
                c_h[ci] = h;
                c_rank[ci] = rank;
                c_lh[ci] = lh;
                const bool big = !BIG && nbr_words(hlen, lh) > arena_words;
                if (big) {  // to the large kernel
                    const uint32_t at = atomicAdd(P.big_count, 1u);
                    P.big_list[at] = item_of(gi, h);
                    P.big_rank[at] = rank;
                    c_lh[ci] = 0;
                }
                // the lists hold h itself once per member
                c_off[ci] = P.emit_entries && c_lh[ci] ? lh - hlen : 0;
            }
        }
        __syncthreads();
        if (tid == 0 && P.emit_entries) {
            uint64_t sum = 0;
            for (uint32_t ci = 0; ci < nc; ci++) sum += c_off[ci];
            uint64_t at = sum ? atomicAdd((unsigned long long*)P.n_entries, (unsigned long long)sum) : 0;
            for (uint32_t ci = 0; ci < nc; ci++) {
                const uint64_t w = c_off[ci];
                c_off[ci] = at;
                at += w;
            }
        }
        __syncthreads();
        for (uint32_t ci = 0; ci < nc; ci++) {
        const uint32_t lh = c_lh[ci];
        if (!lh) continue;  // nothing to do, or the large kernel's
        const HeGraph& G = P.M.graphs[c_gi[ci]];
        const uint32_t h = c_h[ci], rank = c_rank[ci], hlen = G.g.h_len[h], cap = hash_cap(lh);
        const uint64_t hoff = G.g.h_off[h], ebase = c_off[ci];
        uint32_t* keys = arena;
        uint32_t* vals = arena + cap;
        uint32_t* pre = arena + arena_words - (3 * hlen + 4);
        uint64_t* voff = (uint64_t*)(pre + ((hlen + 2) & ~1u));
        if (((uintptr_t)voff & 7) != 0) voff = (uint64_t*)((uint32_t*)voff + 1);
        if (tid == 0) sh.K = 0;
        if (tid < (int)OWN) own[tid] = 0;
        (void)member_prefix(G.g, hoff, hlen, pre, voff, sh.ws);
        for (uint32_t s = tid; s < cap; s += HGT_WG) { keys[s] = HGT_EMPTY; vals[s] = 0; }
        __syncthreads();
        build_nh(G.g, h, hlen, lh, pre, voff, keys, vals, cap, P.in_window != 0, G.window);
        __syncthreads();
        uint32_t* hd = G.hpool + 2 * hoff;
        for (uint32_t s0 = 0; s0 < cap; s0 += HGT_WG) {
            const uint32_t s = s0 + tid;
            const uint32_t x = s < cap ? ld_at<BIG>(&keys[s]) : HGT_EMPTY;
            uint32_t at = 0;
            if (P.emit_entries) {
                const uint64_t m = __ballot(x != HGT_EMPTY);
                if (lane == 0 && m) at = atomicAdd(&sh.K, (uint32_t)__popcll(m));
                at = __shfl(at, 0, 64) + __popcll(m & ((1ull << lane) - 1));
            }
            if (x == HGT_EMPTY) continue;
            const uint32_t c = ld_at<BIG>(&vals[s]);
            const uint32_t fd = hlen > c ? 1u : 0u;
            if (P.emit_entries) {
                const uint64_t q = ebase + at;
                if (q < P.entries_cap) {
                    P.ent_x[q] = (uint32_t)(G.id_base + x);
                    if (P.ent_d) P.ent_d[q] = h;
                    P.ent_pay[q] = ((uint64_t)rank << 32) | ((uint64_t)c << 1) | fd;
                }
            }
            if (P.inserting) {
                uint32_t lx = G.g.h_len[x];
                const uint32_t w = 2 * (c - 1) + (lx > c ? 1u : 0u);
                if (w < OWN) atomicAdd(&own[w], 1u);
                else atomicAdd(&hd[w], 1u);
                // an inserted neighbour builds its own histogram, this one included
                if ((uint32_t)(G.mark[x] >> 32) != G.epoch)
                    atomicAdd(&G.hpool[2 * G.g.h_off[x] + 2 * (c - 1) + fd], 1u);
            }
        }
        __syncthreads();
        if (P.inserting && tid < (int)OWN && own[tid]) atomicAdd(&hd[tid], own[tid]);
        // neighbours met at several members took one entry: the rest of the range is void
        if (P.emit_entries)
            for (uint64_t q = ebase + sh.K + tid; q < ebase + lh - hlen; q += HGT_WG)
                if (q < P.entries_cap) P.ent_x[q] = HGT_EMPTY;
        __syncthreads();
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(HGT_WG) k_nbr_small(NbrParams P) {
    __shared__ __attribute__((aligned(16))) uint32_t arena[ARENA_S];
    nbr_pass_body<false>(P, arena, ARENA_S);
}

__global__ void __launch_bounds__(HGT_WG) k_nbr_big(NbrParams P) {
    nbr_pass_body<true>(P, P.big_scratch + (uint64_t)blockIdx.x * P.big_words, P.big_words);
}

// clear the histograms of the inserted hyperedges (their blocks may be reused); a wave per centre
__global__ void k_h_clear(Multi M) {
    const int lane = threadIdx.x & 63;
    uint64_t q = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (q >= M.total) return;
    uint32_t gi = multi_graph_of(M, q);
    const HeGraph& G = M.graphs[gi];
    if (*G.status) return;
    uint32_t id = G.centres[q - M.base[gi]];
    uint32_t* hb = G.hpool + 2 * G.g.h_off[id];
    uint32_t w = 2 * G.g.h_len[id];
    for (uint32_t i = lane; i < w; i += 64) hb[i] = 0;
}

// remove the deleted hyperedges from their surviving neighbours' histograms
__global__ void k_h_remove(Multi M, const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                           const uint64_t* __restrict__ ent_pay) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t slot = ent_x[i];
        if (slot == HGT_EMPTY) continue;
        const HeGraph& G = M.graphs[multi_graph_of_id(M, slot)];
        if (*G.status) continue;
        uint32_t x = (uint32_t)(slot - G.id_base);
        if ((uint32_t)(G.mark[x] >> 32) == G.epoch) continue;  // x is deleted too
        uint64_t p = ent_pay[i];
        uint32_t k = (uint32_t)(p >> 1) & 0x7fffffffu, f = (uint32_t)p & 1u;
        atomicSub(&G.hpool[2 * G.g.h_off[x] + 2 * (k - 1) + f], 1u);
    }
}

// counting sort of the entries by ID slot: per-slot counts, then scatter
// Entries per ID; with ent_k also an entry's place among its ID's, which saves the scatter
// an atomic that it has to wait for, and the copy of the offsets that the atomics ate.  BL_U
// entries of a thread are in flight together.  Bound by the scattered writes of 8 bytes
// (100k changes on 2M hyperedges, both phases: scatter 1.52 -> 0.66 ms, without the 4 bytes
// that name the changed hyperedge; count 0.85 -> 0.86).
constexpr int BL_U = 4;
__global__ void k_bl_count(const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                           uint64_t* bl_cnt, uint32_t* ent_k) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += BL_U * step) {
        uint32_t x[BL_U];
        uint64_t k[BL_U];
#pragma unroll
        for (int u = 0; u < BL_U; u++) x[u] = i0 + u * step < n ? ent_x[i0 + u * step] : HGT_EMPTY;
        if (!ent_k) {
#pragma unroll
            for (int u = 0; u < BL_U; u++)
                if (x[u] != HGT_EMPTY) atomicAdd((unsigned long long*)&bl_cnt[x[u]], 1ull);
            continue;
        }
#pragma unroll
        for (int u = 0; u < BL_U; u++)
            if (x[u] != HGT_EMPTY) k[u] = atomicAdd((unsigned long long*)&bl_cnt[x[u]], 1ull);
#pragma unroll
        for (int u = 0; u < BL_U; u++)
            if (x[u] != HGT_EMPTY) ent_k[i0 + u * step] = (uint32_t)k[u];
    }
}

__global__ void k_bl_scatter(const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                             const uint32_t* __restrict__ ent_d, const uint64_t* __restrict__ ent_pay,
                             uint64_t* bl_cur, uint32_t* out_d, uint64_t* out_pay) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        if (ent_x[i] == HGT_EMPTY) continue;
        uint64_t pos = atomicAdd((unsigned long long*)&bl_cur[ent_x[i]], 1ull);
        out_d[pos] = ent_d[i];
        out_pay[pos] = ent_pay[i];
    }
}

__global__ void k_bl_place(const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                           const uint32_t* __restrict__ ent_k, const uint64_t* __restrict__ ent_pay,
                           const uint64_t* __restrict__ bl_off, uint64_t* __restrict__ out_pay) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += BL_U * step) {
        uint32_t x[BL_U], k[BL_U];
        uint64_t pay[BL_U], at[BL_U];
#pragma unroll
        for (int u = 0; u < BL_U; u++) {
            const uint64_t i = i0 + u * step;
            x[u] = HGT_EMPTY;
            if (i < n) {
                x[u] = ent_x[i];
                k[u] = ent_k[i];
                pay[u] = ent_pay[i];
            }
        }
#pragma unroll
        for (int u = 0; u < BL_U; u++)
            if (x[u] != HGT_EMPTY) at[u] = bl_off[x[u]];
#pragma unroll
        for (int u = 0; u < BL_U; u++)
            if (x[u] != HGT_EMPTY) out_pay[at[u] + k[u]] = pay[u];
    }
}

// the entry buffer is sized for the worst case; overflow is an internal error of every graph
__global__ void k_entries_check(Multi M, const uint64_t* n_entries_p, uint64_t cap) {
    if (*n_entries_p <= cap) return;
    for (uint32_t g = threadIdx.x; g < M.n_graphs; g += blockDim.x)
        atomicCAS(const_cast<int32_t*>(M.graphs[g].status), 0, HGT_EDEVICE);
}

// ===========================================================================
// the delta kernel
// ===========================================================================
// Stage 0 takes its centres from the batch, keeps every table in 24 KB of LDS and moves
// the centres that do not fit to list 0.  Stage 1 takes list 0 with 54 KB of LDS, stage 2
// (the global stage) list 1 with its tables in a slice of global memory per workgroup and
// the counters in LDS; there a centre with many pairs is shared by several workgroups
// (slices), each of which builds the tables and takes its share of the neighbours.  What
// does not fit there either goes to list 2, which feeds the 2-hop kernel.

// Counters of the class changes of the workgroup's graph so far (mod 2^64).  Every lane
// of a wave adds to one of few classes, so the counters are kept 16-fold, a copy per
// lane of a row of lanes: adds of one instruction meet at most four to a word.
constexpr int COPIES = 16;
struct He2Acc {
    uint64_t pair[HGT_N_HE_CLASSES * COPIES];
    uint64_t open[8 * COPIES];                 // [hlen > c] << 2 | [x only] << 1 | [y only]
    uint64_t tot[HGT_N_HE_CLASSES];
    uint8_t cls8[8];                           // class of an open path by the same three bits
};

__device__ __forceinline__ void pair_add(He2Acc& A, uint32_t cls, uint64_t v) {
    if (cls < 255)
        atomicAdd((unsigned long long*)&A.pair[cls * COPIES + (threadIdx.x & (COPIES - 1))], (unsigned long long)v);
}

// The same for the temporal classes.
constexpr int TCOPIES = 8;
struct TmpAcc {
    uint64_t pair[HGT_N_TEMPORAL_CLASSES * TCOPIES];
};

__device__ __forceinline__ void tmp_add(TmpAcc& A, int cls, uint64_t v) {
    if (cls < 255)
        atomicAdd((unsigned long long*)&A.pair[cls * TCOPIES + (threadIdx.x & (TCOPIES - 1))], (unsigned long long)v);
}

// A pair of neighbours of h in the window of all three: its class by arrival, and when
// the two meet the open paths h-x-y and h-y-x taken back.
__device__ __forceinline__ void tmp_pair(const GraphView& g, const Tables& T, TmpAcc& A, uint32_t h, uint32_t x, uint32_t y,
                                         int64_t th, int64_t tx, int64_t ty, uint32_t hlen, uint32_t mx, uint32_t my,
                                         uint32_t s, uint32_t shh) {
    uint64_t qh = 0, qx = 0, qy = 0;
    if (tx == ty || tx == th || ty == th) {  // only ties need the arrival sequence
        qh = g.h_seq[h];
        qx = g.h_seq[x];
        qy = g.h_seq[y];
    }
    const int nh = (int)hlen, nx = (int)meta_len(mx), ny = (int)meta_len(my), hx = (int)meta_c(mx), hy = (int)meta_c(my);
    tmp_add(A, T.tmp[time_code(th, qh, tx, qx, ty, qy, nh, nx, ny, hx, (int)s, hy, (int)shh)], 1);
    if (!s) return;
    tmp_add(A, T.tmp[time_code(th, qh, tx, qx, ty, qy, nh, nx, ny, hx, (int)s, 0, 0)], ~0ull);
    tmp_add(A, T.tmp[time_code(th, qh, tx, qx, ty, qy, nh, nx, ny, 0, (int)s, hy, 0)], ~0ull);
}
template <int WG>
__device__ __forceinline__ void he2_flush_graph(const He2Params& P, uint32_t g, TmpAcc& A) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < HGT_N_TEMPORAL_CLASSES; i += WG) {
        uint64_t s = 0;
        for (int c = 0; c < TCOPIES; c++) {
            s += A.pair[i * TCOPIES + c];
            A.pair[i * TCOPIES + c] = 0;
        }
        if (g != 0xffffffffu && s) atomicAdd((unsigned long long*)&P.M.graphs[g].out_tmp[i], (unsigned long long)s);
    }
    __syncthreads();
}

// Adds the workgroup's counts to graph g's phase accumulators and clears them.
template <int WG>
__device__ __forceinline__ void he2_flush_graph(const He2Params& P, uint32_t g, He2Acc& A) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < HGT_N_HE_CLASSES * COPIES; i += WG) {
        if (A.pair[i]) atomicAdd((unsigned long long*)&A.tot[i / COPIES], (unsigned long long)A.pair[i]);
        A.pair[i] = 0;
    }
    for (uint32_t i = threadIdx.x; i < 8 * COPIES; i += WG) {
        const uint32_t c = A.cls8[i / COPIES];
        if (A.open[i] && c < 255) atomicAdd((unsigned long long*)&A.tot[c], (unsigned long long)A.open[i]);
        A.open[i] = 0;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < HGT_N_HE_CLASSES; i += WG) {
        if (g != 0xffffffffu && A.tot[i])
            atomicAdd((unsigned long long*)&P.M.graphs[g].out_he[i], (unsigned long long)A.tot[i]);
        A.tot[i] = 0;
    }
    __syncthreads();
}

// Exclusive prefix over i of f(i), i < n, by the whole workgroup: every wave takes
// a contiguous part (one reduce pass, one scan pass, one barrier between them).
// put(i, before) stores the prefix.  Ends without a barrier.
template <int WG, int U, class F, class S>
__device__ __forceinline__ void wg_prefix(uint32_t n, uint32_t* ws, F f, S put) {
    constexpr uint32_t NW = WG / 64;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t per = ((n + NW * 64 - 1) / (NW * 64)) * 64;
    const uint32_t b = wave * per < n ? wave * per : n, e = b + per < n ? b + per : n;
    uint32_t sum = 0;
    for (uint32_t i0 = b; i0 < e; i0 += 64 * U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = i0 + 64 * u + lane < e ? f(i0 + 64 * u + lane) : 0;
#pragma unroll
        for (int u = 0; u < U; u++) sum += v[u];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) ws[wave] = sum;
    __syncthreads();
    uint32_t base = 0;
    for (uint32_t w = 0; w < wave; w++) base += ws[w];
    for (uint32_t i0 = b; i0 < e; i0 += 64 * U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = i0 + 64 * u + lane < e ? f(i0 + 64 * u + lane) : 0;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t i = i0 + 64 * u + lane;
            uint32_t inc = v[u];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(inc, o, 64);
                if (lane >= (uint32_t)o) inc += t;
            }
            if (i < e) put(i, base + inc - v[u]);
            base += __shfl(inc, 63, 64);
        }
    }
}

// N(h) -> c_x in the hash keys/vals, from the lists of h's members.
template <int WG, bool TMP>
__device__ __forceinline__ void he2_nh(const GraphView& G, uint32_t h, uint32_t hlen, uint32_t lh, const uint32_t* pre,
                                       const uint64_t* voff, uint32_t* keys, uint32_t* vals, uint32_t cap, int64_t w_lo,
                                       int64_t w_hi) {
    for (uint32_t s = threadIdx.x; s < cap; s += WG) { keys[s] = HGT_EMPTY; vals[s] = 0; }
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < lh; p += WG) {
        const uint32_t k = seg_of<uint32_t>(pre, hlen, p);
        const uint64_t at = voff[k] + (p - pre[k]);
        const uint32_t x = G.v2h[at];
        if (TMP) {
            const int64_t t = G.v2h_ts[at];
            if (t < w_lo || t > w_hi) continue;
        }
        if (x != h) (void)fr_add(keys, vals, cap, x, 1u);
    }
    __syncthreads();
}

// The hash's neighbours as numbers 0 .. K-1: ID and meta (c | len << 14 | eligible
// << 28 | h < x << 29), and the words of their rows.
template <int WG, bool GLOBAL>
__device__ __forceinline__ void he2_compact(const He2Params& P, const HeGraph& G, Sh2& sh, const uint32_t* keys,
                                            const uint32_t* vals, uint32_t cap, uint32_t* nl_x, uint32_t* nl_meta) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t lens = 0;
    for (uint32_t s0 = 0; s0 < cap; s0 += WG) {
        const uint32_t s = s0 + threadIdx.x;
        const uint32_t x = s < cap ? ld_at<GLOBAL>(&keys[s]) : HGT_EMPTY;
        const uint64_t m = __ballot(x != HGT_EMPTY);
        if (!m) continue;
        uint32_t q = 0;
        if (lane == 0) q = atomicAdd(&sh.K, (uint32_t)__popcll(m));
        q = __shfl(q, 0, 64) + __popcll(m & ((1ull << lane) - 1));
        if (x == HGT_EMPTY) continue;
        const uint32_t c = ld_at<GLOBAL>(&vals[s]), len = G.g.h_len[x];
        const bool elig = P.static_mode || !lower_ranked_member(G.mark[x], G.epoch, sh.rank);
        nl_x[q] = x;
        nl_meta[q] = c | (len << 14) | ((uint32_t)elig << 28) | ((sh.h < x ? 1u : 0u) << 29);
        lens += len;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lens += __shfl_xor(lens, o, 64);
    if (lane == 0) atomicAdd(&sh.rows, lens);
    __syncthreads();
}

// Disjoint-pair classes of all eligible neighbour pairs, from a histogram over
// (f = [|x| > c], c): every pair of neighbours as if x and y were disjoint.
// cnt: 2 (hlen + 1) LDS words.
template <int WG>
__device__ __forceinline__ void he2_disjoint(Sh2& sh, const Tables& T, He2Acc& A, const uint32_t* nl_meta, uint32_t K, uint32_t hlen,
                             uint32_t* cnt) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, Wc = hlen + 1;
    for (uint32_t i = tid; i < 2 * Wc; i += WG) cnt[i] = 0;
    if (tid < 8) sh.g[tid] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < K; i += WG) {
        const uint32_t m = nl_meta[i];
        if (meta_elig(m)) atomicAdd(&cnt[(meta_len(m) > meta_c(m) ? Wc : 0) + meta_c(m)], 1u);
    }
    __syncthreads();
    // inclusive prefix over c of each half, one wave a half
    if (tid < 128) {
        uint32_t* row = cnt + (tid >> 6) * Wc;
        uint32_t base = 0;
        for (uint32_t i0 = 0; i0 < Wc; i0 += 64) {
            const uint32_t i = i0 + lane;
            uint32_t inc = i < Wc ? row[i] : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(inc, o, 64);
                if (lane >= (uint32_t)o) inc += t;
            }
            if (i < Wc) row[i] = base + inc;
            base += __shfl(inc, 63, 64);
        }
    }
    __syncthreads();
    // n_f(c) neighbours with c_x = c; S_f(k) of them with c_x >= k.  Pairs with
    // c_x + c_y >= |h| leave nothing of h alone.
    const uint64_t N0 = cnt[hlen], N1 = cnt[Wc + hlen];
    uint64_t g00 = 0, g01 = 0, g11 = 0, d0 = 0, d1 = 0;
    for (uint32_t c = 1 + tid; c <= hlen; c += WG) {
        const uint64_t n0 = cnt[c] - cnt[c - 1], n1 = cnt[Wc + c] - cnt[Wc + c - 1];
        const uint32_t k = hlen - c;
        const uint64_t s0 = N0 - (k ? cnt[k - 1] : 0), s1 = N1 - (k ? cnt[Wc + k - 1] : 0);
        g00 += n0 * s0;
        g01 += n0 * s1;
        g11 += n1 * s1;
        if (2 * c >= hlen) { d0 += n0; d1 += n1; }
    }
    if (g00 | g01 | g11 | d0 | d1) {
        atomicAdd((unsigned long long*)&sh.g[0], (unsigned long long)g00);
        atomicAdd((unsigned long long*)&sh.g[1], (unsigned long long)g01);
        atomicAdd((unsigned long long*)&sh.g[2], (unsigned long long)g11);
        atomicAdd((unsigned long long*)&sh.g[3], (unsigned long long)d0);
        atomicAdd((unsigned long long*)&sh.g[4], (unsigned long long)d1);
    }
    __syncthreads();
    if (tid == 0) {
        const uint64_t G00 = (sh.g[0] - sh.g[3]) / 2, G11 = (sh.g[2] - sh.g[4]) / 2, G01 = sh.g[1];
        const uint64_t T00 = N0 * (N0 - (N0 ? 1 : 0)) / 2, T11 = N1 * (N1 - (N1 ? 1 : 0)) / 2, T01 = N0 * N1;
        acc_add(A.tot, T.he[40 | 1], T00 - G00);
        acc_add(A.tot, T.he[40], G00);
        acc_add(A.tot, T.he[40 | 4 | 1], T01 - G01);
        acc_add(A.tot, T.he[40 | 4], G01);
        acc_add(A.tot, T.he[40 | 6 | 1], T11 - G11);
        acc_add(A.tot, T.he[40 | 6], G11);
    }
}

// Open paths h - x - y through the histograms of up to 64 neighbours (lane l: ID x, meta m,
// take: eligible and this workgroup's), by one wave: histograms and batch-neighbour lists
// laid end to end.
__device__ __forceinline__ void he2_open(const He2Params& P, const HeGraph& G, const Sh2& sh, He2Acc& A, Flat& F,
                                         uint32_t* wm, uint64_t* woff, bool take, uint32_t x, uint32_t m, uint64_t* st) {
    const uint32_t hlen = sh.hlen, lane = threadIdx.x & 63;
    auto add = [&](uint32_t c, uint32_t k, uint32_t lx, uint32_t f, uint64_t v) {
        // k = |x & y|: x has a vertex outside h and y when k < |x| - c
        const uint32_t i = (hlen > c ? 4u : 0u) | (k < lx - c ? 2u : 0u) | f;
        atomicAdd((unsigned long long*)&A.open[i * COPIES + (lane & (COPIES - 1))], (unsigned long long)v);
    };
    uint32_t lx = 0, bn = 0;
    uint64_t bo = 0;
    if (take) {
        lx = meta_len(m);
        bo = P.bl_off[G.id_base + x];
        bn = (uint32_t)P.bl_cnt[G.id_base + x];
        woff[lane] = G.g.h_off[x];
        // the histogram holds h itself: k = c, y only = |h| > c
        const uint32_t c = meta_c(m);
        add(c, c, lx, hlen > c ? 1u : 0u, ~0ull);
        if (P.stats)  // x's histogram, list bounds and batch-neighbour entries
            atomicAdd((unsigned long long*)&st[1], (unsigned long long)(8ull * lx + 16 + 8ull * bn));
    }
    wm[lane] = m;
    const uint64_t* H = (const uint64_t*)G.hpool;
    wave_flat<4>(F, lx, [&](uint32_t l, uint32_t r) { return H[woff[l] + r]; },
                 [&](bool ok, uint32_t l, uint32_t r, uint32_t, uint64_t hh) {
                     if (!ok || !hh) return;
                     const uint32_t ml = wm[l];
                     if ((uint32_t)hh) add(meta_c(ml), r + 1, meta_len(ml), 0, (uint32_t)hh);
                     if (hh >> 32) add(meta_c(ml), r + 1, meta_len(ml), 1, hh >> 32);
                 });
    // minus every lower-ranked batch member adjacent to x (the pair phase leaves out the
    // ones that meet h)
    woff[lane] = bo;
    wave_flat<4>(F, bn, [&](uint32_t l, uint32_t r) { return P.bl_pay[woff[l] + r]; },
                 [&](bool ok, uint32_t l, uint32_t, uint32_t, uint64_t pay) {
                     if (!ok || (uint32_t)(pay >> 32) >= sh.rank) return;
                     const uint32_t ml = wm[l];
                     add(meta_c(ml), (uint32_t)(pay >> 1) & 0x7fffffffu, meta_len(ml), (uint32_t)pay & 1u, ~0ull);
                 });
}

// The class changes of n intersecting neighbour pairs of one kind (|x & y| = s,
// |h & x & y| = shh), both eligible: in a full count the closed triad at its smallest-ID
// centre, in a delta the open paths h-x-y and h-y-x taken back and the true class in place
// of the disjoint one.
__device__ __forceinline__ void he2_pair(const He2Params& P, const Tables& T, He2Acc& A, uint32_t hlen, uint32_t mx,
                                         uint32_t my, uint32_t s, uint32_t shh, uint64_t n) {
    const uint32_t xl = meta_len(mx), yl = meta_len(my), cx = meta_c(mx), cy = meta_c(my);
    const uint32_t cf = (hlen > cx + cy ? 1u : 0u) | (xl > cx ? 2u : 0u) | (yl > cy ? 4u : 0u) | 40u;
    const uint32_t ct = (hlen + shh > cx + cy ? 1u : 0u) | (xl + shh > cx + s ? 2u : 0u) | (yl + shh > cy + s ? 4u : 0u) |
                        (cx > shh ? 8u : 0u) | (s > shh ? 16u : 0u) | (cy > shh ? 32u : 0u) | (shh ? 64u : 0u);
    pair_add(A, T.he[cf], 0 - n);
    if (P.static_mode) {
        if ((mx & my) >> 29 & 1u) pair_add(A, T.he[ct], n);
        return;
    }
    pair_add(A, T.he[ct], n);
    pair_add(A, A.cls8[(hlen > cx ? 4u : 0u) | (xl > cx + s ? 2u : 0u) | (yl > s ? 1u : 0u)], 0 - n);
    pair_add(A, A.cls8[(hlen > cy ? 4u : 0u) | (yl > cy + s ? 2u : 0u) | (xl > s ? 1u : 0u)], 0 - n);
}

// Pairs of neighbours that meet inside h, as if they met nowhere else.  What a pair
// changes depends on x only through its mask of shared members, min(|x| - c, c + 1) and
// (in a full count) h < x, so neighbours are counted by these and the pairs taken by kind:
// a few dozen kinds in place of hundreds of neighbours.  One workgroup does it for a centre, also
// for one in slices: where every neighbour is a kind of its own, 2,000 neighbours that share 12
// of a centre's 64 members take 7.7 ms in all, 6,000 of 6 members 70 (the 2-hop kernel: 92 and
// 97).  rep/cnt: gcap slots, list: K words.
template <int WG, bool BIG, bool GLOBAL>
__device__ __forceinline__ void he2_kinds(const He2Params& P, Sh2& sh, const Tables& T, He2Acc& A, const uint32_t* nl_meta,
                          const uint32_t* mask, uint32_t K, uint32_t hlen, uint32_t* rep, uint32_t gcap) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t* cnt = rep + gcap;
    uint32_t* list = cnt + gcap;
    auto mask_of = [&](uint32_t i) {
        return (uint64_t)ld_at<BIG>(&mask[2 * i]) | (uint64_t)ld_at<BIG>(&mask[2 * i + 1]) << 32;
    };
    auto rest_of = [&](uint32_t m) {
        const uint32_t c = meta_c(m), d = meta_len(m) - c;
        return (d < c + 1 ? d : c + 1) | (P.static_mode ? m & (1u << 29) : 0u);
    };
    for (uint32_t s = tid; s < gcap; s += WG) { rep[s] = HGT_EMPTY; cnt[s] = 0; }
    if (tid == 0) sh.G = 0;
    __syncthreads();
    for (uint32_t i = tid; i < K; i += WG) {
        const uint32_t m = nl_meta[i];
        if (!meta_elig(m)) continue;
        const uint64_t mk = mask_of(i);
        const uint32_t rs = rest_of(m);
        uint32_t s = fr_slot((uint32_t)mk * 0x9e3779b1u ^ (uint32_t)(mk >> 32) * 0x85ebca6bu ^ rs * 0xc2b2ae35u, gcap);
        for (uint32_t probe = 0; probe < gcap; probe++) {
            const uint32_t r = atomicCAS(&rep[s], HGT_EMPTY, i);
            if (r == HGT_EMPTY) list[atomicAdd(&sh.G, 1u)] = s;
            if (r == HGT_EMPTY || (mask_of(r) == mk && rest_of(nl_meta[r]) == rs)) {
                atomicAdd(&cnt[s], 1u);
                break;
            }
            s = fr_next(s, gcap);
        }
    }
    __syncthreads();
    const uint32_t Gn = sh.G;
    for (uint32_t a = wave; a < Gn; a += WG / 64) {
        const uint32_t sa = list[a], ra = ld_at<GLOBAL>(&rep[sa]), na = ld_at<GLOBAL>(&cnt[sa]), ma = nl_meta[ra];
        const uint64_t ka = mask_of(ra);
        for (uint32_t b = a + lane; b < Gn; b += 64) {
            const uint32_t sb = list[b], rb = ld_at<GLOBAL>(&rep[sb]);
            const uint32_t shh = __popcll(ka & mask_of(rb));
            if (!shh) continue;
            const uint64_t n = a == b ? (uint64_t)na * (na - 1) / 2 : (uint64_t)na * ld_at<GLOBAL>(&cnt[sb]);
            if (n) he2_pair(P, T, A, hlen, ma, nl_meta[rb], shh, shh, n);
        }
    }
    __syncthreads();
}

template <int STAGE, int WG, bool TMP>
__device__ __forceinline__ void he2_body(const He2Params& P, uint32_t* arena, const uint32_t AW, uint32_t* lds, Sh2& sh, const Tables& T,
                         std::conditional_t<TMP, TmpAcc, He2Acc>& A, uint64_t* st, uint64_t* ph) {
    constexpr uint32_t NW = WG / 64;
    constexpr bool BIG = STAGE == 2, SLICED = STAGE > 0;
    constexpr uint32_t BM_LOG = BIG ? 17 : STAGE ? 15 : 14;  // bits of each vertex bitmap
    constexpr uint32_t BH_LOG = 12, BH_WORDS = 1u << (BH_LOG - 5);  // ... and of the one of h's members
    constexpr uint32_t BM_WORDS = 1u << (BM_LOG - 5);
    constexpr uint32_t POS = 0x7fffffffu;               // a run cursor; the top bit: the vertex lies in h
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ Flat flat[NW];
    __shared__ uint64_t woff_all[NW][64];
    __shared__ uint32_t wm_all[NW][64];
    Flat& fl = flat[wave];
    uint64_t* woff = woff_all[wave];
    uint32_t* wm = wm_all[wave];
    uint32_t q = 0, q_end = 0;  // thread 0: work items taken
    uint64_t t_mark = 0;    // thread 0: wall clock at the last phase mark (profiling)
    uint64_t t_centre = 0;  // ... at the start of the current centre
#define HE2_MARK(i)                                     \
    do {                                                \
        if (P.phase_ticks && tid == 0) {                \
            uint64_t t_ = wall_clock64();               \
            ph[i] += t_ - t_mark;                       \
            t_mark = t_;                                \
        }                                               \
    } while (0)
    for (;;) {
        if (tid == 0) {
            const uint64_t n = !SLICED ? P.M.total : P.slice_pre[P.slice_cap + 1];
            if (q == q_end) {
                const uint32_t take = take_size(n, gridDim.x);
                q = atomicAdd(&P.queue[STAGE], take);
                q_end = q + take;
            }
            const uint32_t c = q++;
            sh.stop = c >= n;
            sh.slice = 0;
            sh.nslice = 1;
            if (!sh.stop) {
                uint32_t gi, h, rank;
                if (!SLICED) {
                    gi = multi_graph_of(P.M, c);
                    rank = (uint32_t)(c - P.M.base[gi]);
                    h = P.M.graphs[gi].centres[rank];
                } else {  // slice c of the centres' slices
                    const uint32_t nc = (uint32_t)P.slice_pre[P.slice_cap];
                    const uint32_t ci = seg_of<uint64_t>(P.slice_pre, nc, c);
                    const uint64_t at = P.slice_pre[ci], next = ci + 1 < nc ? P.slice_pre[ci + 1] : n;
                    sh.slice = (uint32_t)(c - at);
                    sh.nslice = (uint32_t)(next - at);
                    const uint64_t it = P.list[STAGE - 1][ci];
                    gi = (uint32_t)(it >> 32);
                    h = (uint32_t)it;
                    rank = P.rank[STAGE - 1][ci];
                }
                const HeGraph& Gq = P.M.graphs[gi];
                sh.gi = gi;
                sh.h = h;
                sh.rank = rank;
                sh.skip = *((volatile const int32_t*)Gq.status) != 0;
                sh.hlen = Gq.g.h_len[h];
                sh.hoff = Gq.g.h_off[h];
                sh.defer = (3ull * sh.hlen + 4 > (BIG ? LDS_L : AW / 2) || STAGE < P.force_stage) ? 1u : 0u;
                sh.K = sh.W = sh.S = sh.rows = 0;
            }
        }
        __syncthreads();
        if (sh.stop) break;
        if (P.phase_ticks && tid == 0) t_mark = t_centre = wall_clock64();
        if (sh.gi != sh.cur_g) {  // the counts so far belong to the previous graph
            he2_flush_graph<WG>(P, sh.cur_g, A);
            if (tid == 0) sh.cur_g = sh.gi;
            __syncthreads();
        }
        if (sh.skip) {
            __syncthreads();
            continue;
        }
        const HeGraph& G = P.M.graphs[sh.gi];
        const uint32_t h = sh.h, hlen = sh.hlen, slice = sh.slice, nslice = sh.nslice;
        // a centre that does not fit moves on whole: its first slice puts it on the list
        auto move_on = [&]() {
            if (tid == 0 && slice == 0) {
                const uint32_t q = atomicAdd(&P.count[STAGE], 1u);
                P.list[STAGE][q] = item_of(sh.gi, h);
                P.rank[STAGE][q] = sh.rank;
                atomicAdd((unsigned long long*)&st[0], 1ull);
            }
            HE2_MARK(7);
            __syncthreads();
        };
        if (sh.defer) {
            move_on();
            continue;
        }
        // --- members of h: degree prefix and list offsets, in LDS (at the arena's end in stage 0)
        uint32_t* pre = BIG ? lds : arena + AW - (3 * hlen + 4);
        uint64_t* voff = (uint64_t*)(pre + ((hlen + 2) & ~1u));
        if (((uintptr_t)voff & 7) != 0) voff = (uint64_t*)((uint32_t*)voff + 1);
        wg_prefix<WG, 1>(hlen, sh.ws,
                      [&](uint32_t i) {
                          const uint32_t m = G.g.h2v[sh.hoff + i];
                          voff[i] = G.g.v_off[m];
                          return G.g.v_len[m];
                      },
                      [&](uint32_t i, uint32_t b) { pre[i] = b; });
        __syncthreads();
        if (tid == 0) {
            uint32_t lh = 0;
            for (uint32_t w = 0; w < NW; w++) lh += sh.ws[w];
            pre[hlen] = lh;
            sh.lh = lh;
            const uint64_t cap = (uint64_t)lh + lh / 2 + 32;
            sh.defer = (lh >= K_MAX_N || 2 * cap + (TMP ? 4ull : 2ull) * lh + 4 * hlen + 8 > AW) ? 1u : 0u;
        }
        __syncthreads();
        if (sh.defer) {
            move_on();
            continue;
        }
        HE2_MARK(0);
        // --- N(h).  Arena: hash (2 cap), later the masks of shared members | IDs and metas of
        // the neighbours (lh each) | h's members
        const uint32_t lh = sh.lh, cap = hash_cap(lh);
        uint32_t* mask = arena;
        uint32_t* nl_x = arena + 2 * cap;
        uint32_t* nl_meta = nl_x + lh;
        int64_t* nl_t = (int64_t*)(nl_meta + lh);  // 2 cap and 2 lh are even
        uint32_t* hm = nl_meta + (TMP ? 3 * lh : lh);
        uint32_t base0 = (uint32_t)(hm + hlen - arena);
        const int64_t th = TMP ? G.g.h_ts[h] : 0, w_lo = ts_sub(th, G.window), w_hi = ts_add(th, G.window);
        const uint32_t lds_used = BIG ? (3 * hlen + 8) & ~1u : 0;  // pre and voff
        if (BIG && lds_used + 2 * cap <= LDS_L) {
            he2_nh<WG, TMP>(G.g, h, hlen, lh, pre, voff, lds + lds_used, lds + lds_used + cap, cap, w_lo, w_hi);
            HE2_MARK(1);
            he2_compact<WG, false>(P, G, sh, lds + lds_used, lds + lds_used + cap, cap, nl_x, nl_meta);
        } else {
            he2_nh<WG, TMP>(G.g, h, hlen, lh, pre, voff, arena, arena + cap, cap, w_lo, w_hi);
            HE2_MARK(1);
            he2_compact<WG, BIG>(P, G, sh, arena, arena + cap, cap, nl_x, nl_meta);
        }
        HE2_MARK(2);
        const uint32_t K = sh.K, per = K / NW + 1 < 64 ? K / NW + 1 : 64;
        const bool masked = hlen <= MASK_BITS;
        if (TMP)
            for (uint32_t i = tid; i < K; i += WG) nl_t[i] = G.g.h_ts[nl_x[i]];
        // --- vertices outside h that two neighbours may share: a second row holding a vertex
        // finds its bit set and sets the bit in the second bitmap (the members are stashed, so a
        // row is gathered once).  Members of h (a third bitmap tells) go into the neighbour's
        // mask; with more members than a mask holds they are treated like the others.
        uint32_t* row_at = arena + base0;  // K words: the rows' places in the stash
        uint32_t* ecnt = row_at + K;       // K words: shared vertices of each neighbour
        base0 += 2 * K;
        uint32_t* bm = BIG ? lds : arena + base0;
        uint32_t* bh = bm + 2 * BM_WORDS;
        uint32_t* hs = BIG ? bh + BH_WORDS : hm;  // looked through where bh has a bit: with masks only
        static_assert(!BIG || 2 * BM_WORDS + BH_WORDS + MASK_BITS <= LDS_L, "global stage LDS");
        uint32_t* stash = arena + base0 + (BIG ? 0 : 2 * BM_WORDS + BH_WORDS);
        const uint32_t stash0 = (uint32_t)(stash - arena);
        const uint32_t room = stash0 < AW ? AW - stash0 : 0;
        // rows that do not fit are not gathered: a quarter of the centres of a power-law graph
        // leave stage 0 here (100k changes on 2M hyperedges, left after the gather: stage 0 4.30
        // -> 3.96 ms, stage 1 3.53 -> 3.38)
        if (!room || sh.rows > room) {
            move_on();
            continue;
        }
        for (uint32_t i = tid; i < 2 * BM_WORDS + BH_WORDS; i += WG) bm[i] = 0;
        if (masked)
            for (uint32_t i = tid; i < 2 * K; i += WG) mask[i] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < hlen; i += WG) {
            const uint32_t v = G.g.h2v[sh.hoff + i], b = (v * 2654435761u) >> (32 - BH_LOG);
            hm[i] = v;
            if (BIG && masked) hs[i] = v;
            if (masked) atomicOr(&bh[b >> 5], 1u << (b & 31));
        }
        __syncthreads();
        // a wave's chunks of neighbours: rows [c0, c0 + n)
        auto chunks = [&](auto fn) __attribute__((always_inline)) {
            for (uint32_t c0 = wave * per; c0 < K; c0 += NW * per) fn(c0, K - c0 < per ? K - c0 : per);
        };
        chunks([&](uint32_t c0, uint32_t n) {
            uint32_t d = 0;
            if (lane < n) {
                d = meta_len(nl_meta[c0 + lane]);
                woff[lane] = G.g.h_off[nl_x[c0 + lane]];
            }
            const FlatSeg g = flat_lay(fl, d);
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&sh.W, g.tot);
            base = __builtin_amdgcn_readfirstlane(base);
            if (lane < n) row_at[c0 + lane] = base + g.ex;
            for (uint32_t w0 = 0; w0 < g.tot; w0 += 4096) {
                flat_window(fl, g, w0);
                flat_walk<4>(fl, g, w0, [&](uint32_t l, uint32_t r) { return G.g.h2v[woff[l] + r]; },
                    [&](bool ok, uint32_t l, uint32_t, uint32_t p, uint32_t v) {
                        if (!ok) return;
                        const uint32_t hv = v * 2654435761u, bj = hv >> (32 - BH_LOG);
                        uint32_t in = 0;
                        if (bh[bj >> 5] >> (bj & 31) & 1u) {
                            const uint32_t k = lower_bound_u32(hs, hlen, v);
                            if (k < hlen && hs[k] == v) {
                                in = 1u << 31;
                                atomicOr(&mask[2 * (c0 + l) + (k >> 5)], 1u << (k & 31));
                            }
                        }
                        if (base + p < room) stash[base + p] = v | in;
                        if (in) return;
                        const uint32_t b = hv >> (32 - BM_LOG), bit = 1u << (b & 31);
                        if (atomicOr(&bm[b >> 5], bit) & bit) atomicOr(&bm[BM_WORDS + (b >> 5)], bit);
                    });
                wave_sync();
            }
        });
        __syncthreads();
        const uint32_t W = sh.W;
        if (tid == 0) {
            // h's row and its members' incidence lists, each neighbour's row and metadata
            if (P.stats)
                atomicAdd((unsigned long long*)&st[1], (unsigned long long)(4ull * (hlen + lh) + 20ull * K + 4ull * W));
        }
        // Walks the stashed rows, d(xi) entries of each, and packs what keep() wants to the front
        // of its row (a row belongs to one wave, which has read what it writes over): keep(c0, ok,
        // l, v) puts new values in place of PU entries, of neighbours c0 + l, HGT_EMPTY to drop
        // them.  ecnt: the entries left.
        constexpr int PU = 4;
        auto pack = [&](auto dfn, auto keep) __attribute__((always_inline)) {
            uint32_t left = 0;
            chunks([&](uint32_t c0, uint32_t n) {
                uint32_t d = 0;
                if (lane < n) {
                    d = dfn(c0 + lane);
                    woff[lane] = row_at[c0 + lane];
                }
                wm[lane] = 0;
                const FlatSeg g = flat_lay(fl, d);
                for (uint32_t w0 = 0; w0 < g.tot; w0 += 4096) {
                    flat_window(fl, g, w0);
                    flat_walk_all<PU>(fl, g, w0, [&](uint32_t l, uint32_t r) { return stash[woff[l] + r]; },
                                      [&](const bool (&ok)[PU], const uint32_t (&l)[PU], uint32_t (&v)[PU]) {
                                          keep(c0, ok, l, v);
#pragma unroll
                                          for (int u = 0; u < PU; u++)
                                              if (v[u] != HGT_EMPTY) stash[woff[l[u]] + atomicAdd(&wm[l[u]], 1u)] = v[u];
                                      });
                    wave_sync();
                }
                wave_sync();
                if (lane < n) {
                    ecnt[c0 + lane] = wm[lane];
                    left += wm[lane];
                }
                wave_sync();
            });
            return left;
        };
        {
            const uint32_t left = pack([&](uint32_t i) { return meta_len(nl_meta[i]); },
                                       [&](uint32_t, const bool (&ok)[PU], const uint32_t (&)[PU], uint32_t (&v)[PU]) {
#pragma unroll
                                           for (int u = 0; u < PU; u++) {
                                               const uint32_t b = (v[u] * 2654435761u) >> (32 - BM_LOG);
                                               if (!ok[u] || v[u] >> 31 || !(bm[BM_WORDS + (b >> 5)] >> (b & 31) & 1u))
                                                   v[u] = HGT_EMPTY;
                                           }
                                       });
            if (left) atomicAdd(&sh.S, left);
        }
        __syncthreads();
        const uint32_t S = sh.S;
        // --- exact groups: a hash of the vertices that are left, their runs, and per neighbour
        // the slots of those that another one holds too.  The regions go where they fit: over the
        // bitmaps, after the stash, or over the hash of N(h).
        uint32_t lo_at = masked ? 2 * K : 0, bm_at = base0, hi_at = stash0 + W;
        const uint32_t lo_end = 2 * cap, bm_end = stash0;
        bool fits = true;
        auto place = [&](uint32_t words) -> uint32_t {
            uint32_t r = 0;
            if (lo_at + words <= lo_end) { r = lo_at; lo_at += words; }
            else if (bm_at + words <= bm_end) { r = bm_at; bm_at += words; }
            else if (hi_at + words <= AW) { r = hi_at; hi_at += words; }
            else fits = false;
            return r;
        };
        const uint32_t vcap = hash_cap(S < G.n_vertices ? S : G.n_vertices);
        // the counters; before them the (c, f) histogram and the kinds of neighbours
        const uint32_t gcap = hash_cap(K), k_words = masked && !TMP ? 2 * gcap + K : 0;
        const uint32_t cw = BIG ? CNT_L : K / 4 + 16;  // counter words per wave
        uint32_t c_words = NW * cw > 2 * hlen + 2 ? NW * cw : 2 * hlen + 2;
        if (k_words > c_words) c_words = k_words;
        uint32_t* rx = arena + place(S);
        uint32_t* tst = arena + place(vcap + 1);  // the vertices, then the runs' starts
        uint32_t* tcnt = arena + place(vcap);
        uint32_t* cnts = BIG ? lds : arena + place(c_words);
        const bool k_lds = !BIG || k_words <= LDS_L;
        uint32_t* kinds = k_lds ? cnts : arena + place(k_words);
        if (!fits) {
            __syncthreads();
            move_on();
            continue;
        }
        HE2_MARK(4);
        if (S) {
            for (uint32_t s = tid; s < vcap; s += WG) { tst[s] = HGT_EMPTY; tcnt[s] = 0; }
            __syncthreads();
            // all entries' probes are in flight together: in the global stage each is a trip to the L2
            (void)pack([&](uint32_t i) { return ecnt[i]; },
                       [&](uint32_t, const bool (&ok)[PU], const uint32_t (&)[PU], uint32_t (&v)[PU]) {
                           if constexpr (!BIG) {
#pragma unroll
                               for (int u = 0; u < PU; u++) v[u] = ok[u] ? fr_add(tst, tcnt, vcap, v[u], 1u) : HGT_EMPTY;
                               return;
                           }
                           uint32_t s[PU], k[PU];
                           uint32_t go = 0;
#pragma unroll
                           for (int u = 0; u < PU; u++) {
                               s[u] = fr_slot(v[u], vcap);
                               go |= ok[u] ? 1u << u : 0u;
                           }
                           for (uint32_t probe = 0; go && probe < vcap; probe++) {
#pragma unroll
                               for (int u = 0; u < PU; u++) k[u] = ld_at<BIG>(&tst[s[u]]);
#pragma unroll
                               for (int u = 0; u < PU; u++)
                                   if (k[u] == HGT_EMPTY && (go >> u & 1u)) k[u] = atomicCAS(&tst[s[u]], HGT_EMPTY, v[u]);
#pragma unroll
                               for (int u = 0; u < PU; u++) {
                                   if (k[u] == HGT_EMPTY || k[u] == v[u]) go &= ~(1u << u);
                                   else if (go >> u & 1u) s[u] = fr_next(s[u], vcap);
                               }
                           }
#pragma unroll
                           for (int u = 0; u < PU; u++) {
                               if (ok[u]) atomicAdd(&tcnt[s[u]], 1u);
                               v[u] = ok[u] ? s[u] : HGT_EMPTY;
                           }
                       });
            __syncthreads();
            // run starts (vertices of one neighbour only: an empty run), flagged when the vertex lies in h
            wg_prefix<WG, BIG ? 4 : 1>(vcap, sh.ws,
                          [&](uint32_t s) {
                              const uint32_t r = ld_at<BIG>(&tcnt[s]);
                              return r >= 2 ? r : 0u;
                          },
                          [&](uint32_t s, uint32_t b) {
                              uint32_t in = 0;
                              if (!masked) {
                                  const uint32_t v = ld_at<BIG>(&tst[s]);
                                  in = v != HGT_EMPTY && contains_u32(hm, hlen, v) ? 1u << 31 : 0;
                              }
                              tst[s] = b | in;
                          });
            if (tid == 0) {  // the end of the last run
                uint32_t t = 0;
                for (uint32_t w = 0; w < NW; w++) t += sh.ws[w];
                tst[vcap] = t;
            }
            __syncthreads();
            (void)pack([&](uint32_t i) { return ecnt[i]; },
                       [&](uint32_t c0, const bool (&ok)[PU], const uint32_t (&l)[PU], uint32_t (&v)[PU]) {
                           if constexpr (!BIG) {
#pragma unroll
                               for (int u = 0; u < PU; u++) {
                                   if (!ok[u]) { v[u] = HGT_EMPTY; continue; }
                                   const uint32_t s0 = tst[v[u]] & POS, s1 = tst[v[u] + 1] & POS;
                                   if (s0 == s1) v[u] = HGT_EMPTY;
                                   else rx[s0 + atomicSub(&tcnt[v[u]], 1u) - 1] = c0 + l[u];
                               }
                               return;
                           }
                           uint32_t r0[PU], r1[PU];
#pragma unroll
                           for (int u = 0; u < PU; u++) {
                               const uint32_t s = ok[u] ? v[u] : 0;
                               r0[u] = ld_at<BIG>(&tst[s]) & POS;
                               r1[u] = ld_at<BIG>(&tst[s + 1]) & POS;
                           }
#pragma unroll
                           for (int u = 0; u < PU; u++) {
                               if (!ok[u] || r0[u] == r1[u]) v[u] = HGT_EMPTY;
                               else r0[u] += atomicSub(&tcnt[v[u]], 1u) - 1;
                           }
#pragma unroll
                           for (int u = 0; u < PU; u++)
                               if (v[u] != HGT_EMPTY) rx[r0[u]] = c0 + l[u];
                       });
        }
        __syncthreads();
        // now neighbour i's shared vertices are the slots stash[row_at[i] .. + ecnt[i]) and the
        // neighbours at slot s rx[tst[s] .. tst[s + 1])
        HE2_MARK(8);
        // --- disjoint-pair classes (the first slice); the histogram lies over the counters in the global stage
        if constexpr (!TMP) {
            if (slice == 0) {
                he2_disjoint<WG>(sh, T, A, nl_meta, K, hlen, cnts);
                __syncthreads();
                if (masked) {
                    if (k_lds) he2_kinds<WG, BIG, false>(P, sh, T, A, nl_meta, mask, K, hlen, cnts, gcap);
                    else he2_kinds<WG, BIG, true>(P, sh, T, A, nl_meta, mask, K, hlen, kinds, gcap);
                }
            }
        }
        __syncthreads();
        HE2_MARK(3);
        // --- open paths h - x - y through the histograms, per eligible neighbour
        if constexpr (!TMP)
            for (uint32_t c0 = P.static_mode ? K : wave * per; c0 < K; c0 += NW * per) {
                uint32_t x = 0, m = 0;
                bool take = lane < per && c0 + lane < K;
                if (take) {
                    x = nl_x[c0 + lane];
                    m = nl_meta[c0 + lane];
                    take = meta_elig(m) && (nslice == 1 || slice_of(x, nslice) == slice);
                }
                he2_open(P, G, sh, A, fl, wm, woff, take, x, m, st);
            }
        HE2_MARK(5);
        // --- intersecting neighbour pairs (masked: those that meet outside h too)
        auto mask_of = [&](uint32_t i) {
            return (uint64_t)ld_at<BIG>(&mask[2 * i]) | (uint64_t)ld_at<BIG>(&mask[2 * i + 1]) << 32;
        };
        uint32_t* cnt = cnts + wave * cw;
        for (uint32_t i = lane; i < cw; i += 64) cnt[i] = 0;
        wave_sync();
        // a wave's neighbours are every NW-th, looked at 64 at a time.  The slices of a centre
        // number its neighbours each in its own order, so a row belongs to the slice that its ID
        // names and a pair to its row of smaller ID; unsliced, a pair belongs to its earlier row.
        for (uint32_t c0 = 0; c0 * NW < K; c0 += 64) {
          const uint32_t il = wave + NW * (c0 + lane);
          uint32_t mx_l = 0, e0_l = 0, n_l = 0, x_l = 0;
          if (il < K) {
              mx_l = nl_meta[il];
              e0_l = row_at[il];
              n_l = S ? ecnt[il] : 0;
              if (nslice > 1) x_l = nl_x[il];
          }
          uint64_t rows = __ballot(il < K && meta_elig(mx_l) && (TMP || n_l) &&
                                   (nslice == 1 || slice_of(x_l, nslice) == slice));
          // the runs of a row's (first 64) shared vertices, fetched a row ahead
          auto fetch = [&](int r, uint32_t from, uint32_t& at, uint32_t& len) __attribute__((always_inline)) {
              const uint32_t e = from + lane;
              len = 0;
              if (e < (uint32_t)__builtin_amdgcn_readlane(n_l, r)) {
                  const uint32_t s = stash[__builtin_amdgcn_readlane(e0_l, r) + e];
                  at = ld_at<BIG>(&tst[s]);
                  len = (ld_at<BIG>(&tst[s + 1]) & POS) - (at & POS);
              }
          };
          uint32_t at_n = 0, len_n = 0;
          if (rows) fetch(__ffsll((unsigned long long)rows) - 1, 0, at_n, len_n);
          while (rows) {
            const int r = __ffsll((unsigned long long)rows) - 1;
            rows &= rows - 1;
            const uint32_t at_c = at_n, len_c = len_n;
            if (rows) fetch(__ffsll((unsigned long long)rows) - 1, 0, at_n, len_n);
            const uint32_t i = wave + NW * (c0 + r);
            const uint32_t mx = __builtin_amdgcn_readlane(mx_l, r), ne = __builtin_amdgcn_readlane(n_l, r);
            const uint32_t x = __builtin_amdgcn_readlane(x_l, r);
            const uint64_t mkx = masked ? mask_of(i) : 0;
            const int64_t tx = TMP ? nl_t[i] : 0;
            // counters of a word by what they can reach: bytes (or two, |x & y| and |h & x & y|
            // without a mask) for rows of up to 255 members
            const uint32_t lw = meta_len(mx) > 255 ? 0 : masked ? 2 : 1, bits = 32u >> lw;
            const uint32_t cm = 0xffffffffu >> (32 - bits), half = 16u >> lw, win = cw << lw;
            FlatSeg g{0, 0, 0};
            const bool one = ne <= 64;
            if (one && ne) {
                wm[lane] = at_c;
                g = flat_lay(fl, len_c);
                if (g.tot <= 4096) flat_window(fl, g, 0);
            }
            // every neighbour on the runs of x's shared vertices: fn(y, [the vertex lies in h])
            auto walk = [&](auto fn) __attribute__((always_inline)) {
                auto load = [&](uint32_t l, uint32_t j) { return rx[(wm[l] & POS) + j]; };
                auto use = [&](bool ok, uint32_t l, uint32_t, uint32_t, uint32_t y) {
                    if (ok) fn(y, wm[l] >> 31);
                };
                if (one && g.tot <= 4096) {
                    flat_walk<4>(fl, g, 0, load, use);
                    return;
                }
                for (uint32_t e = 0; e < ne; e += 64) {
                    uint32_t at = 0, len = 0;
                    fetch(r, e, at, len);
                    wave_sync();
                    wm[lane] = at;
                    (void)wave_flat<4>(fl, len, load, use);
                }
            };
            for (uint32_t w0 = nslice == 1 ? i + 1 : 0; w0 < K; w0 += win) {
                const uint32_t w1 = K - w0 < win ? K : w0 + win;
                if (ne)
                    walk([&](uint32_t y, uint32_t in) {
                        if (y >= w0 && y < w1)
                            atomicAdd(&cnt[(y - w0) >> lw], (masked ? 1u : 1u + (in << half)) << (((y - w0) & ((1u << lw) - 1)) * bits));
                    });
                wave_sync();
                auto take = [&](uint32_t y, uint32_t v) __attribute__((always_inline)) {
                    if (nslice > 1 && nl_x[y] <= x) return;  // the other row's
                    const uint32_t my = nl_meta[y];
                    if (!meta_elig(my)) return;
                    // masked: v vertices outside h, on top of those inside
                    const uint32_t shh = masked ? (uint32_t)__popcll(mkx & mask_of(y)) : v >> half;
                    const uint32_t sxy = masked ? shh + v : v & ((1u << half) - 1);
                    if constexpr (TMP) {
                        const int64_t ty = nl_t[y];
                        if (within(th, tx, ty, G.window))
                            tmp_pair(G.g, T, A, h, nl_x[i], nl_x[y], th, tx, ty, hlen, mx, my, sxy, shh);
                    } else {
                        he2_pair(P, T, A, hlen, mx, my, sxy, shh, 1);
                        if (masked && shh) he2_pair(P, T, A, hlen, mx, my, shh, shh, ~0ull);
                    }
                };
                // the counted ones, by a look at all counters or by another walk, whichever is shorter
                // (temporal: every pair of neighbours has a class of its own)
                const uint32_t words = (w1 - w0 + (1u << lw) - 1) >> lw;
                if (TMP) {
                    for (uint32_t y = w0 + lane; y < w1; y += 64)
                        take(y, ne ? cnt[(y - w0) >> lw] >> (((y - w0) & ((1u << lw) - 1)) * bits) & cm : 0);
                    wave_sync();
                    if (ne)
                        for (uint32_t k = lane; k < words; k += 64) cnt[k] = 0;
                } else if (words <= 2 * g.tot + 64) {
                    for (uint32_t k = lane; k < words; k += 64) {
                        const uint32_t c = cnt[k];
                        if (!c) continue;
                        cnt[k] = 0;
                        for (uint32_t b = 0; b < 1u << lw; b++) {
                            const uint32_t v = c >> (b * bits) & cm;
                            if (v) take(w0 + (k << lw) + b, v);
                        }
                    }
                } else {
                    walk([&](uint32_t y, uint32_t) {
                        if (y < w0 || y >= w1) return;
                        const uint32_t sft = ((y - w0) & ((1u << lw) - 1)) * bits;
                        const uint32_t v = atomicAnd(&cnt[(y - w0) >> lw], ~(cm << sft)) >> sft & cm;
                        if (v) take(y, v);  // else taken at another shared vertex
                    });
                }
                wave_sync();
            }
          }
        }
        __syncthreads();
        HE2_MARK(6);
        // the longest centre this workgroup finished (slot HE2_PHASES - 1 holds a maximum)
        if (P.phase_ticks && tid == 0 && t_mark - t_centre > ph[HE2_PHASES - 1]) ph[HE2_PHASES - 1] = t_mark - t_centre;
    }
#undef HE2_MARK
}

template <int STAGE>
__device__ __forceinline__ void he2_flush_stats(const He2Params& P, const uint64_t* st, const uint64_t* ph) {
    if (P.phase_ticks && threadIdx.x < HE2_PHASES - 1 && ph[threadIdx.x])
        atomicAdd((unsigned long long*)&P.stats[ST_PH0 + HE2_PHASES * STAGE + threadIdx.x],
                  (unsigned long long)ph[threadIdx.x]);
    if (P.phase_ticks && threadIdx.x == HE2_PHASES - 1 && ph[threadIdx.x])
        atomicMax((unsigned long long*)&P.stats[ST_PH0 + HE2_PHASES * STAGE + threadIdx.x],
                  (unsigned long long)ph[threadIdx.x]);
    if (P.stats && threadIdx.x == 0 && st[0])
        atomicAdd((unsigned long long*)&P.stats[ST_DEFER0 + STAGE], (unsigned long long)st[0]);
    if (P.stats && threadIdx.x == 0 && st[1])
        atomicAdd((unsigned long long*)&P.stats[ST_HEB0 + STAGE], (unsigned long long)st[1]);
}

template <int STAGE, int WG, bool TMP>
__device__ __forceinline__ void he2_kernel(const He2Params& P, uint32_t* arena, uint32_t words, uint32_t* lds) {
    __shared__ Sh2 sh;
    __shared__ Tables T;
    __shared__ std::conditional_t<TMP, TmpAcc, He2Acc> A;
    __shared__ uint64_t st[2];
    __shared__ uint64_t ph[HE2_PHASES];
    const uint32_t tid = threadIdx.x;
    if (tid < HE2_PHASES) ph[tid] = 0;
    if (tid == 0) sh.cur_g = 0xffffffffu;
    if constexpr (TMP) {
        for (uint32_t i = tid; i < 128; i += WG) T.tmp[i] = P.tmp_tab[i];
        for (uint32_t i = tid; i < HGT_N_TEMPORAL_CLASSES * TCOPIES; i += WG) A.pair[i] = 0;
    } else {
        for (uint32_t i = tid; i < 128; i += WG) T.he[i] = P.he_tab[i];
        for (uint32_t i = tid; i < HGT_N_HE_CLASSES * COPIES; i += WG) A.pair[i] = 0;
        for (uint32_t i = tid; i < 8 * COPIES; i += WG) A.open[i] = 0;
        if (tid < HGT_N_HE_CLASSES) A.tot[tid] = 0;
        // open path: h & x (8) and x & y (16), h only (1), x only (2), y only (4)
        if (tid < 8) A.cls8[tid] = P.he_tab[24 | (tid & 4 ? 1 : 0) | (tid & 2 ? 2 : 0) | (tid & 1 ? 4 : 0)];
    }
    if (tid < 2) st[tid] = 0;
    __syncthreads();
    he2_body<STAGE, WG, TMP>(P, arena, words, lds, sh, T, A, st, ph);
    he2_flush_graph<WG>(P, sh.cur_g, A);
    if constexpr (!TMP) he2_flush_stats<STAGE>(P, st, ph);
    else if (P.stats && tid == 0)
        atomicAdd((unsigned long long*)&P.stats[ST_BYTES_BIG], (unsigned long long)st[1]);
}

#define HE2_STAGES(NAME, TMP)                                                                                   \
    __global__ void __launch_bounds__(HGT_WG, 4) NAME##_s0(He2Params P) {                                       \
        __shared__ __attribute__((aligned(16))) uint32_t arena[ARENA_S];                                        \
        he2_kernel<0, HGT_WG, TMP>(P, arena, ARENA_S, nullptr);                                                 \
    }                                                                                                           \
    __global__ void __launch_bounds__(WG_M, 4) NAME##_s1(He2Params P) {                                         \
        __shared__ __attribute__((aligned(16))) uint32_t arena[ARENA_M];                                        \
        he2_kernel<1, WG_M, TMP>(P, arena, ARENA_M, nullptr);                                                   \
    }                                                                                                           \
    __global__ void __launch_bounds__(WG_W, 4) NAME##_s1w(He2Params P) {                                        \
        __shared__ __attribute__((aligned(16))) uint32_t arena[ARENA_W];                                        \
        he2_kernel<1, WG_W, TMP>(P, arena, ARENA_W, nullptr);                                                   \
    }                                                                                                           \
    __global__ void __launch_bounds__(WG_L, 4) NAME##_s2(He2Params P) {                                         \
        __shared__ __attribute__((aligned(16))) uint32_t lds[LDS_L];                                            \
        he2_kernel<2, WG_L, TMP>(P, P.garena + (uint64_t)blockIdx.x * P.garena_words, (uint32_t)P.garena_words, \
                                 lds);                                                                          \
    }
HE2_STAGES(k_he2, false)
HE2_STAGES(k_tmp, true)
#undef HE2_STAGES

// Slices of the centres of stages 1 and 2.  A wave per centre estimates its work in walked
// run entries: its lists (the rows are gathered by every slice), and the pairs of its
// neighbours.  Those that meet inside h count when h is too long for masks (squares of the
// list lengths); outside h, a vertex of degree d lies in about d K / E neighbours, so the
// runs' squares sum to (K / E)^2 sum_v d^2, and sum_v d^2 is the incidences times the
// degree of a random member, for which h's own members stand in.
__global__ void k_he2_work(Multi M, const uint64_t* __restrict__ list, const uint32_t* n_p, uint64_t cap,
                           uint32_t slice_lh, int tmp, uint64_t* pre, uint64_t* total) {
    const int lane = threadIdx.x & 63;
    const uint32_t n = *n_p;
    uint64_t sum = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) pre[cap] = n;
    for (uint64_t c = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; c < n;
         c += ((uint64_t)gridDim.x * blockDim.x) >> 6) {
        const uint64_t it = list[c];
        const HeGraph& G = M.graphs[(uint32_t)(it >> 32)];
        const GraphView& g = G.g;
        const uint32_t h = (uint32_t)it;
        const uint32_t* row = g.h2v + g.h_off[h];
        const uint32_t len = g.h_len[h];
        uint64_t lh = 0, sq = 0;
        for (uint32_t i = lane; i < len; i += 64) {
            const uint64_t d = g.v_len[row[i]];
            lh += d;
            sq += d * d;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lh += __shfl_xor(lh, o, 64);
            sq += __shfl_xor(sq, o, 64);
        }
        double w = (double)lh * (double)lh * G.pair_scale * ((double)lh / (len ? len : 1));
        const double all = (double)lh * (double)lh;
        if (w > all) w = all;
        if (len > MASK_BITS) w += (double)sq;
        if (tmp) w += all / 16;  // every pair in the window has a class of its own
        w += 32.0 * (double)lh;
        const uint64_t work = slice_lh ? (lh + slice_lh - 1) / slice_lh : (uint64_t)w;
        if (lane == 0) pre[c] = work;
        sum += work;
    }
    if (lane == 0 && sum) atomicAdd((unsigned long long*)total, (unsigned long long)sum);
}

// Work to slices, and their exclusive prefix, by one workgroup.  A slice holds about a
// workgroup's share of the whole where there are few centres, half of one where there are
// several per workgroup, so that the last ones end together: every slice builds its
// centre's tables again, which for 500 dense centres, one per workgroup, is most of the
// work (a quarter of a share each: 7.4 ms; this rule: 5.1; all centres whole: 5.4), while
// 3,300 centres of uneven size gain by being cut (6.5 ms whole, 5.9 so).
constexpr uint64_t SLICE_MIN = 1ull << 15;
constexpr uint32_t SLICES_MAX = 64;
__global__ void __launch_bounds__(1024) k_he2_cut(uint64_t cap, uint32_t slice_lh, uint64_t slice_pairs, uint32_t grid,
                                                  const uint64_t* total, uint64_t* pre) {
    __shared__ uint32_t ws[16];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t n = pre[cap];
    const uint64_t shares = n / 2 < grid ? grid : n / 2 < 2ull * grid ? n / 2 : 2ull * grid;
    uint64_t per = *total / shares;
    if (per < SLICE_MIN) per = SLICE_MIN;
    if (slice_pairs) per = slice_pairs;
    uint64_t base = 0;
    for (uint64_t b = 0; b < n; b += 1024) {
        const uint64_t c = b + threadIdx.x;
        uint32_t sl = 0;
        if (c < n) {
            const uint64_t w = slice_lh ? pre[c] : (pre[c] + per / 2) / per;
            sl = w < 1 ? 1 : w > SLICES_MAX ? SLICES_MAX : (uint32_t)w;
        }
        uint32_t inc = sl;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(inc, o, 64);
            if (lane >= (uint32_t)o) inc += t;
        }
        if (lane == 63) ws[wave] = inc;
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (uint32_t w = 0; w < 16; w++) {
            if (w < wave) before += ws[w];
            all += ws[w];
        }
        if (c < n) pre[c] = base + before + inc - sl;
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) pre[cap + 1] = base;
}

}  // namespace

void he2_nbr_launch(NbrParams& P, unsigned grid_small, unsigned grid_big, hipStream_t s) {
    hgt_fill_u32(P.queue, 0, 3, s);
    hgt_fill_u64(P.n_entries, 0, 1, s);
    if (P.M.total == 0) return;
    if (P.inserting) k_h_clear<<<(unsigned)((P.M.total * 64 + 255) / 256), 256, 0, s>>>(P.M);
    k_nbr_small<<<grid_small, HGT_WG, 0, s>>>(P);
    k_nbr_big<<<grid_big, HGT_WG, 0, s>>>(P);
    k_entries_check<<<1, 256, 0, s>>>(P.M, P.n_entries, P.entries_cap);
}

void he2_lists_build(NbrParams& P, uint64_t* bl_cnt, uint64_t* bl_off, uint64_t* bl_cur, uint32_t* bl_d,
                     uint64_t* bl_pay, void* scan_tmp, hipStream_t s) {
    const uint64_t n_ids = P.M.total_ids;
    hgt_fill_u64(bl_cnt, 0, n_ids, s);
    unsigned g = 2048;
    // who an entry came from matters to the temporal paths only; without, its place takes the column
    uint32_t* ent_k = P.ent_d ? nullptr : P.ent_k;
    k_bl_count<<<g, 256, 0, s>>>(P.n_entries, P.entries_cap, P.ent_x, bl_cnt, ent_k);
    hgt_scan_u64(bl_cnt, bl_off, n_ids, nullptr, nullptr, scan_tmp, s);
    if (ent_k) {
        k_bl_place<<<g, 256, 0, s>>>(P.n_entries, P.entries_cap, P.ent_x, ent_k, P.ent_pay, bl_off, bl_pay);
        return;
    }
    (void)hipMemcpyAsync(bl_cur, bl_off, n_ids * 8, hipMemcpyDeviceToDevice, s);
    k_bl_scatter<<<g, 256, 0, s>>>(P.n_entries, P.entries_cap, P.ent_x, P.ent_d, P.ent_pay, bl_cur, bl_d, bl_pay);
}

void he2_remove_deleted(NbrParams& P, hipStream_t s) {
    if (P.M.total == 0) return;
    k_h_remove<<<2048, 256, 0, s>>>(P.M, P.n_entries, P.entries_cap, P.ent_x, P.ent_pay);
}

namespace {

// Stages 1 and 2: each cuts the centres that the stage before moved on.
void launch_sliced(He2Params& P, int stage, unsigned grid, bool wide, bool tmp, hipStream_t s) {
    if (!P.M.total) return;
    const uint64_t cap = P.slice_cap;
    const unsigned waves = (unsigned)((cap + 3) / 4);
    uint64_t* total = P.work_total + (stage - 1);
    k_he2_work<<<waves < 1024 ? waves : 1024, 256, 0, s>>>(P.M, P.list[stage - 1], &P.count[stage - 1], cap, P.slice_lh,
                                                           tmp ? 1 : 0, P.slice_pre, total);
    k_he2_cut<<<1, 1024, 0, s>>>(cap, P.slice_lh, P.slice_pairs, grid, total, P.slice_pre);
    if (stage == 1 && wide) {
        if (tmp) k_tmp_s1w<<<grid, WG_W, 0, s>>>(P);
        else k_he2_s1w<<<grid, WG_W, 0, s>>>(P);
    } else if (stage == 1) {
        if (tmp) k_tmp_s1<<<grid, WG_M, 0, s>>>(P);
        else k_he2_s1<<<grid, WG_M, 0, s>>>(P);
    } else {
        if (tmp) k_tmp_s2<<<grid, WG_L, 0, s>>>(P);
        else k_he2_s2<<<grid, WG_L, 0, s>>>(P);
    }
}

}  // namespace

void he2_launch_lds(He2Params& P, unsigned grid, unsigned grid_mid, bool wide, hipStream_t s) {
    if (P.M.total) k_he2_s0<<<grid, HGT_WG, 0, s>>>(P);
    launch_sliced(P, 1, grid_mid, wide, false, s);
}
void he2_launch_global(He2Params& P, unsigned grid, hipStream_t s) { launch_sliced(P, 2, grid, false, false, s); }

void tmp_launch_lds(He2Params& P, unsigned grid, unsigned grid_mid, bool wide, hipStream_t s) {
    if (P.M.total) k_tmp_s0<<<grid, HGT_WG, 0, s>>>(P);
    launch_sliced(P, 1, grid_mid, wide, true, s);
}
void tmp_launch_global(He2Params& P, unsigned grid, hipStream_t s) { launch_sliced(P, 2, grid, false, true, s); }
