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
// Neighbour pairs {x, y} of h that intersect get their true class in place of
// the disjoint-pair class that the histogram pass gave them.  They are found
// along the runs of the vertices that two or more neighbours share: a wave
// takes a neighbour x, walks the runs of x's shared vertices and counts
// |x & y| and |h & x & y| for every later neighbour y in a table of LDS counters
// indexed by the neighbour's number (no hashing, no sort), then walks the runs
// again, taking each y's counter as it empties it.
#include "triad_common.h"

namespace {

using namespace tri;

constexpr uint32_t ARENA_S = 7168;     // stage 0: 28 KB of LDS, 256 threads, four workgroups per CU
constexpr int WG_L = 512;              // global stage: threads per workgroup
constexpr uint32_t CNT_L = 2048;       // ... counters per wave: neighbours are taken in windows of this many
constexpr uint32_t LDS_L = 16640;      // ... LDS words: counters of 8 waves, or two bitmaps, or a (c, f) histogram
static_assert(LDS_L >= (WG_L / 64) * CNT_L && LDS_L >= 2 * (HGT_MAX_CARD + 1), "global stage LDS");
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

struct Sh2 {
    uint32_t h, rank, hlen, lh, K, W, S, defer, stop, over;
    uint32_t gi, cur_g, skip;
    uint32_t slice, nslice;
    uint64_t hoff;
    uint32_t ws[WG_L / 64];
    uint32_t ncap;
    uint64_t g[8];
};

// ---- per-centre neighbourhood (shared by the neighbour pass and the delta kernel)
// Builds N(h) -> c_x in the hash at keys/vals (already cleared), reading the
// incidence lists of h's members through pre/voff.
__device__ __forceinline__ void build_nh(const GraphView& G, uint32_t h, uint32_t hlen, uint32_t lh, const uint32_t* pre,
                                         const uint64_t* voff, uint32_t* keys, uint32_t* vals, uint32_t cap) {
    for (uint32_t p = threadIdx.x; p < lh; p += HGT_WG) {
        uint32_t k = seg_of<uint32_t>(pre, hlen, p);
        uint32_t x = G.v2h[voff[k] + (p - pre[k])];
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
template <bool BIG>
__device__ void nbr_pass_body(const NbrParams& P, uint32_t* arena, uint64_t arena_words) {
    __shared__ Sh2 sh;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) {
            uint64_t n = BIG ? (uint64_t)*P.big_count : P.M.total;
            uint32_t c = atomicAdd(BIG ? P.big_queue : P.queue, 1u);
            sh.stop = c >= n;
            if (!sh.stop) {
                uint32_t gi, h, rank;
                if (BIG) {
                    uint64_t it = P.big_list[c];
                    gi = (uint32_t)(it >> 32);
                    h = (uint32_t)it;
                    rank = P.big_rank[c];
                } else {
                    gi = multi_graph_of(P.M, c);
                    rank = (uint32_t)(c - P.M.base[gi]);
                    h = P.M.graphs[gi].centres[rank];
                }
                const HeGraph& Gq = P.M.graphs[gi];
                sh.gi = gi;
                sh.h = h;
                sh.rank = rank;
                sh.skip = *((volatile const int32_t*)Gq.status) != 0;
                sh.hlen = Gq.g.h_len[h];
                sh.hoff = Gq.g.h_off[h];
                // prefix + offsets must fit at the arena end
                sh.defer = (!BIG && 3ull * sh.hlen + 4 > arena_words / 2) ? 1u : 0u;
            }
        }
        __syncthreads();
        if (sh.stop) break;
        if (sh.skip) {
            __syncthreads();
            continue;
        }
        const HeGraph& G = P.M.graphs[sh.gi];
        if (!sh.defer) {
            const uint32_t hlen = sh.hlen;
            uint32_t* pre = arena + arena_words - (3 * hlen + 4);
            uint64_t* voff = (uint64_t*)(pre + ((hlen + 2) & ~1u));
            if (((uintptr_t)voff & 7) != 0) voff = (uint64_t*)((uint32_t*)voff + 1);
            uint32_t lh = member_prefix(G.g, sh.hoff, hlen, pre, voff, sh.ws);
            uint32_t cap = hash_cap(lh);
            if (tid == 0) {
                sh.lh = lh;
                sh.ncap = cap;
                sh.defer = (!BIG && 2ull * cap + 3ull * hlen + 4 > arena_words) ? 1u : 0u;
            }
            __syncthreads();
        }
        if (sh.defer) {
            if (tid == 0) {
                uint32_t q = atomicAdd(P.big_count, 1u);
                P.big_list[q] = item_of(sh.gi, sh.h);
                P.big_rank[q] = sh.rank;
            }
            __syncthreads();
            continue;
        }
        const uint32_t h = sh.h, hlen = sh.hlen, lh = sh.lh, cap = sh.ncap;
        uint32_t* keys = arena;
        uint32_t* vals = arena + cap;
        uint32_t* pre = arena + arena_words - (3 * hlen + 4);
        uint64_t* voff = (uint64_t*)(pre + ((hlen + 2) & ~1u));
        if (((uintptr_t)voff & 7) != 0) voff = (uint64_t*)((uint32_t*)voff + 1);
        for (uint32_t s = tid; s < cap; s += HGT_WG) { keys[s] = HGT_EMPTY; vals[s] = 0; }
        __syncthreads();
        build_nh(G.g, h, hlen, lh, pre, voff, keys, vals, cap);
        __syncthreads();
        uint32_t* hd = G.hpool + 2 * sh.hoff;
        // the centre's entries take one range of the entry array, reserved at once (one
        // atomic per centre on the shared cursor instead of one per entry)
        if (P.emit_entries) {
            if (tid == 0) sh.K = 0;
            __syncthreads();
            uint32_t mine = 0;
            for (uint32_t s = tid; s < cap; s += HGT_WG) mine += ld_at<BIG>(&keys[s]) != HGT_EMPTY ? 1u : 0u;
            if (mine) atomicAdd(&sh.K, mine);
            __syncthreads();
            if (tid == 0) {
                sh.g[0] = atomicAdd((unsigned long long*)P.n_entries, (unsigned long long)sh.K);
                sh.K = 0;
            }
            __syncthreads();
        }
        const uint64_t ebase = P.emit_entries ? sh.g[0] : 0;
        for (uint32_t s0 = 0; s0 < cap; s0 += HGT_WG) {
            const uint32_t s = s0 + tid;
            const uint32_t x = s < cap ? ld_at<BIG>(&keys[s]) : HGT_EMPTY;
            uint32_t at = 0;
            if (P.emit_entries) {
                const uint64_t m = __ballot(x != HGT_EMPTY);
                if ((tid & 63) == 0 && m) at = atomicAdd(&sh.K, (uint32_t)__popcll(m));
                at = __shfl(at, 0, 64) + __popcll(m & ((1ull << (tid & 63)) - 1));
            }
            if (x == HGT_EMPTY) continue;
            const uint32_t c = ld_at<BIG>(&vals[s]);
            const uint32_t fd = hlen > c ? 1u : 0u;
            if (P.emit_entries) {
                const uint64_t q = ebase + at;
                if (q < P.entries_cap) {
                    P.ent_x[q] = (uint32_t)(G.id_base + x);
                    P.ent_d[q] = h;
                    P.ent_pay[q] = ((uint64_t)sh.rank << 32) | ((uint64_t)c << 1) | fd;
                }
            }
            if (P.inserting) {
                uint32_t lx = G.g.h_len[x];
                atomicAdd(&hd[2 * (c - 1) + (lx > c ? 1u : 0u)], 1u);
                // an inserted neighbour builds its own histogram, this one included
                if ((uint32_t)(G.mark[x] >> 32) != G.epoch)
                    atomicAdd(&G.hpool[2 * G.g.h_off[x] + 2 * (c - 1) + fd], 1u);
            }
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
__global__ void k_bl_count(const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                           uint64_t* bl_cnt) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        atomicAdd((unsigned long long*)&bl_cnt[ent_x[i]], 1ull);
}

__global__ void k_bl_scatter(const uint64_t* n_entries_p, uint64_t cap, const uint32_t* __restrict__ ent_x,
                             const uint32_t* __restrict__ ent_d, const uint64_t* __restrict__ ent_pay,
                             uint64_t* bl_cur, uint32_t* out_d, uint64_t* out_pay) {
    uint64_t n = *n_entries_p;
    if (n > cap) n = cap;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t pos = atomicAdd((unsigned long long*)&bl_cur[ent_x[i]], 1ull);
        out_d[pos] = ent_d[i];
        out_pay[pos] = ent_pay[i];
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
// Stage 0 takes its centres from the batch, keeps every table in 28 KB of LDS and
// moves the centres that do not fit to list 0.  The global stage (stage 2) takes
// list 0 and keeps its tables in a slice of global memory per workgroup, the
// counters in LDS; a centre with many pairs is shared by several workgroups
// (slices), each of which builds the tables and takes every nslice-th neighbour.
// What does not fit there either goes to list 2, which feeds the 2-hop kernel.

// Counters of the class changes of the workgroup's graph so far.  Every lane of
// a wave adds to one of few classes, so the 32-bit pair counters are kept 32-fold
// (a copy per lane pair: adds of one instruction meet at most two to a word) and
// the 64-bit open-path counters too.
constexpr int COPIES = 32;
struct He2Acc {
    uint32_t pair[HGT_N_HE_CLASSES * COPIES];  // signed changes
    uint64_t open[8 * COPIES];                 // [hlen > c] << 2 | [x only] << 1 | [y only]
    uint64_t tot[HGT_N_HE_CLASSES];
    uint8_t cls8[8];                           // class of an open path by the same three bits
    uint8_t pad[8];
};

__device__ __forceinline__ void pair_add(He2Acc& A, uint32_t cls, uint32_t v) {
    if (cls < 255) atomicAdd(&A.pair[cls * COPIES + (threadIdx.x & (COPIES - 1))], v);
}

// Moves the 32-bit counters into the 64-bit totals (any wave, any time).
__device__ __forceinline__ void pair_fold(He2Acc& A) {
    for (uint32_t i = threadIdx.x & 63; i < HGT_N_HE_CLASSES * COPIES; i += 64) {
        const int32_t v = (int32_t)atomicExch(&A.pair[i], 0u);
        if (v) atomicAdd((unsigned long long*)&A.tot[i / COPIES], (unsigned long long)(int64_t)v);
    }
}
constexpr uint32_t FOLD_AT = 1u << 25;  // pairs of one wave after which it folds: no counter passes 2^31

// Adds the workgroup's counts to graph g's phase accumulators and clears them.
template <int WG>
__device__ void he2_flush_graph(const He2Params& P, uint32_t g, He2Acc& A) {
    __syncthreads();
    if (threadIdx.x < 64) pair_fold(A);
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
template <int WG, class F, class S>
__device__ __forceinline__ void wg_prefix(uint32_t n, uint32_t* ws, F f, S put) {
    constexpr uint32_t NW = WG / 64;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t per = ((n + NW * 64 - 1) / (NW * 64)) * 64;
    const uint32_t b = wave * per < n ? wave * per : n, e = b + per < n ? b + per : n;
    uint32_t sum = 0;
    for (uint32_t i = b + lane; i < e; i += 64) sum += f(i);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) ws[wave] = sum;
    __syncthreads();
    uint32_t base = 0;
    for (uint32_t w = 0; w < wave; w++) base += ws[w];
    for (uint32_t i0 = b; i0 < e; i0 += 64) {
        const uint32_t i = i0 + lane;
        const uint32_t v = i < e ? f(i) : 0;
        uint32_t inc = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(inc, o, 64);
            if (lane >= (uint32_t)o) inc += t;
        }
        if (i < e) put(i, base + inc - v);
        base += __shfl(inc, 63, 64);
    }
}

// N(h) -> c_x in the hash keys/vals, from the lists of h's members.
template <int WG>
__device__ __forceinline__ void he2_nh(const GraphView& G, uint32_t h, uint32_t hlen, uint32_t lh, const uint32_t* pre,
                                       const uint64_t* voff, uint32_t* keys, uint32_t* vals, uint32_t cap) {
    for (uint32_t s = threadIdx.x; s < cap; s += WG) { keys[s] = HGT_EMPTY; vals[s] = 0; }
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < lh; p += WG) {
        const uint32_t k = seg_of<uint32_t>(pre, hlen, p);
        const uint32_t x = G.v2h[voff[k] + (p - pre[k])];
        if (x != h) (void)fr_add(keys, vals, cap, x, 1u);
    }
    __syncthreads();
}

// The hash's neighbours as numbers 0 .. K-1: ID and meta (c | len << 14 | eligible
// << 28 | h < x << 29).
template <int WG, bool GLOBAL>
__device__ __forceinline__ void he2_compact(const He2Params& P, const HeGraph& G, Sh2& sh, const uint32_t* keys,
                                            const uint32_t* vals, uint32_t cap, uint32_t* nl_x, uint32_t* nl_meta) {
    const uint32_t lane = threadIdx.x & 63;
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
    }
    __syncthreads();
}

// Disjoint-pair classes of all eligible neighbour pairs, from a histogram over
// (f = [|x| > c], c): every pair of neighbours as if x and y were disjoint.
// cnt: 2 (hlen + 1) LDS words.
template <int WG>
__device__ void he2_disjoint(Sh2& sh, const Tables& T, He2Acc& A, const uint32_t* nl_meta, uint32_t K, uint32_t hlen,
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

// Open paths h - x - y of one neighbour x through its histogram.
__device__ __forceinline__ void he2_open(const He2Params& P, const HeGraph& G, const Sh2& sh, He2Acc& A, uint32_t x,
                                         uint32_t m, uint64_t* st) {
    const uint32_t hlen = sh.hlen, c = meta_c(m), lx = meta_len(m);
    const uint32_t thr = lx - c;  // k < thr  <=>  x has a vertex outside h and y
    const uint64_t* H = (const uint64_t*)(G.hpool + 2 * G.g.h_off[x]);  
    const uint64_t xs = G.id_base + x;
    const uint64_t bo = P.bl_off[xs], bn = P.bl_cnt[xs];
    if (P.stats)  // x's histogram, list bounds and batch-neighbour entries
        atomicAdd((unsigned long long*)&st[1], (unsigned long long)(8ull * lx + 16 + 8ull * bn));
    // a_f: neighbours y with |x & y| < thr (x keeps a private vertex), b_f: the rest
    uint64_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    for (uint32_t k = 1; k <= lx; k++) {
        const uint64_t hh = H[k - 1];
        const uint64_t h0 = (uint32_t)hh, h1 = hh >> 32;
        if (k < thr) { a0 += h0; a1 += h1; }
        else { b0 += h0; b1 += h1; }
    }
    // the histogram holds h itself: k = c, y only = |h| > c
    if (c < thr) { if (hlen > c) a1--; else a0--; }
    else { if (hlen > c) b1--; else b0--; }
    // every lower-ranked batch member adjacent to x (the pair phase leaves out
    // the ones that meet h)
    for (uint64_t e = 0; e < bn; e++) {
        const uint64_t pay = P.bl_pay[bo + e];
        if ((uint32_t)(pay >> 32) >= sh.rank) continue;
        const uint32_t k = (uint32_t)(pay >> 1) & 0x7fffffffu, f = (uint32_t)pay & 1u;
        if (k < thr) { if (f) a1--; else a0--; }
        else { if (f) b1--; else b0--; }
    }
    uint64_t* o = A.open + (hlen > c ? 4 * COPIES : 0) + (threadIdx.x & (COPIES - 1));
    if (b0) atomicAdd((unsigned long long*)&o[0], (unsigned long long)b0);
    if (b1) atomicAdd((unsigned long long*)&o[COPIES], (unsigned long long)b1);
    if (a0) atomicAdd((unsigned long long*)&o[2 * COPIES], (unsigned long long)a0);
    if (a1) atomicAdd((unsigned long long*)&o[3 * COPIES], (unsigned long long)a1);
}

// The class changes of one intersecting neighbour pair (|x & y| = s, |h & x & y| =
// shh), both eligible: in a full count the closed triad at its smallest-ID centre, in
// a delta the open paths h-x-y and h-y-x taken back and the true class in place of the
// disjoint one.
__device__ __forceinline__ void he2_pair(const He2Params& P, const Tables& T, He2Acc& A, uint32_t hlen, uint32_t mx,
                                         uint32_t my, uint32_t s, uint32_t shh) {
    const uint32_t xl = meta_len(mx), yl = meta_len(my), cx = meta_c(mx), cy = meta_c(my);
    const uint32_t cf = (hlen > cx + cy ? 1u : 0u) | (xl > cx ? 2u : 0u) | (yl > cy ? 4u : 0u) | 40u;
    const uint32_t ct = (hlen + shh > cx + cy ? 1u : 0u) | (xl + shh > cx + s ? 2u : 0u) | (yl + shh > cy + s ? 4u : 0u) |
                        (cx > shh ? 8u : 0u) | (s > shh ? 16u : 0u) | (cy > shh ? 32u : 0u) | (shh ? 64u : 0u);
    pair_add(A, T.he[cf], ~0u);
    if (P.static_mode) {
        if ((mx & my) >> 29 & 1u) pair_add(A, T.he[ct], 1u);
        return;
    }
    pair_add(A, T.he[ct], 1u);
    pair_add(A, A.cls8[(hlen > cx ? 4u : 0u) | (xl > cx + s ? 2u : 0u) | (yl > s ? 1u : 0u)], ~0u);
    pair_add(A, A.cls8[(hlen > cy ? 4u : 0u) | (yl > cy + s ? 2u : 0u) | (xl > s ? 1u : 0u)], ~0u);
}

// Rows of all neighbours, a wave per 64 of them: per(xi, v, j) for every member v,
// j counting the members of all rows (row_at[xi] + k for neighbour xi's k-th).  first:
// the rows are laid out one after the other (row_at is written, sh.W their total);
// else their members are read back from `stash`, where per() put them.
template <int WG, class F>
__device__ __forceinline__ void he2_rows(const GraphView& G, Sh2& sh, const uint32_t* nl_x, const uint32_t* nl_meta,
                                         uint32_t* row_at, uint32_t K, const uint32_t* stash, uint32_t (*wpre)[65],
                                         uint64_t (*woff)[64], bool first, F per) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t c0 = wave * 64; c0 < K; c0 += WG) {
        const uint32_t cnt = K - c0 < 64 ? K - c0 : 64;
        uint32_t d = 0;
        if (lane < cnt) {
            d = meta_len(nl_meta[c0 + lane]);
            if (first) woff[wave][lane] = G.h_off[nl_x[c0 + lane]];
        }
        uint32_t inc = d;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(inc, o, 64);
            if (lane >= (uint32_t)o) inc += t;
        }
        const uint32_t tot = __shfl(inc, 63, 64);
        uint32_t base = 0;
        if (first) {
            if (lane == 0) base = atomicAdd(&sh.W, tot);
            base = __shfl(base, 0, 64);
            if (lane < cnt) row_at[c0 + lane] = base + inc - d;
        } else {
            base = row_at[c0];
        }
        wpre[wave][lane + 1] = inc;
        if (lane == 0) wpre[wave][0] = 0;
        wave_sync();
        for (uint32_t p = lane; p < tot; p += 64) {
            const uint32_t k = seg_of<uint32_t>(wpre[wave], cnt, p);
            const uint32_t v = first ? G.h2v[woff[wave][k] + (p - wpre[wave][k])] : stash[base + p];
            per(c0 + k, v, base + p);
        }
        wave_sync();
    }
}

template <bool BIG, int WG>
__device__ void he2_body(const He2Params& P, uint32_t* arena, const uint32_t AW, uint32_t* lds, Sh2& sh, const Tables& T,
                         He2Acc& A, uint64_t* st, uint64_t* ph) {
    constexpr uint32_t NW = WG / 64;
    constexpr int STAGE = BIG ? 2 : 0;
    constexpr uint32_t BM_LOG = BIG ? 18 : 14;          // bits of each vertex bitmap
    constexpr uint32_t BM_WORDS = 1u << (BM_LOG - 5);
    constexpr uint32_t POS = 0x7fffffffu;               // a run cursor; the top bit: the vertex lies in h
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ uint32_t wpre[NW][65];
    __shared__ uint64_t woff[NW][64];
    uint32_t q = 0, q_end = 0;  // thread 0: work items taken
    uint32_t folded = 0;    // pairs this wave counted since its last fold
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
            const uint64_t n = !BIG ? P.M.total : P.slice_pre[P.slice_cap + 1];
            if (q == q_end) {
                const uint32_t take = BIG ? 1 : take_size(n, gridDim.x);
                q = atomicAdd(&P.queue[STAGE], take);
                q_end = q + take;
            }
            const uint32_t c = q++;
            sh.stop = c >= n;
            sh.slice = 0;
            sh.nslice = 1;
            if (!sh.stop) {
                uint32_t gi, h, rank;
                if (!BIG) {
                    gi = multi_graph_of(P.M, c);
                    rank = (uint32_t)(c - P.M.base[gi]);
                    h = P.M.graphs[gi].centres[rank];
                } else {  // slice c of the centres' slices
                    const uint32_t nc = (uint32_t)P.slice_pre[P.slice_cap];
                    const uint32_t ci = seg_of<uint64_t>(P.slice_pre, nc, c);
                    const uint64_t at = P.slice_pre[ci], next = ci + 1 < nc ? P.slice_pre[ci + 1] : n;
                    sh.slice = (uint32_t)(c - at);
                    sh.nslice = (uint32_t)(next - at);
                    const uint64_t it = P.list[0][ci];
                    gi = (uint32_t)(it >> 32);
                    h = (uint32_t)it;
                    rank = P.rank[0][ci];
                }
                const HeGraph& Gq = P.M.graphs[gi];
                sh.gi = gi;
                sh.h = h;
                sh.rank = rank;
                sh.skip = *((volatile const int32_t*)Gq.status) != 0;
                sh.hlen = Gq.g.h_len[h];
                sh.hoff = Gq.g.h_off[h];
                sh.defer = (3ull * sh.hlen + 4 > (BIG ? LDS_L : AW / 2) || STAGE < P.force_stage) ? 1u : 0u;
                sh.K = sh.W = sh.S = sh.over = 0;
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
        wg_prefix<WG>(hlen, sh.ws,
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
            sh.defer = (lh >= K_MAX_N || 2 * cap + 3ull * lh + 4 * hlen + 8 > AW) ? 1u : 0u;
        }
        __syncthreads();
        if (sh.defer) {
            move_on();
            continue;
        }
        HE2_MARK(0);
        // --- N(h).  Arena: hash (2 cap) | IDs, metas, row starts of the neighbours (lh each) | h's members
        const uint32_t lh = sh.lh, cap = hash_cap(lh);
        uint32_t* nl_x = arena + 2 * cap;
        uint32_t* nl_meta = nl_x + lh;
        uint32_t* row_at = nl_meta + lh;
        uint32_t* hm = row_at + lh;
        uint32_t base0 = (uint32_t)(hm + hlen - arena);
        const uint32_t lds_used = BIG ? (3 * hlen + 8) & ~1u : 0;  // pre and voff
        if (BIG && lds_used + 2 * cap <= LDS_L) {
            he2_nh<WG>(G.g, h, hlen, lh, pre, voff, lds + lds_used, lds + lds_used + cap, cap);
            HE2_MARK(1);
            he2_compact<WG, false>(P, G, sh, lds + lds_used, lds + lds_used + cap, cap, nl_x, nl_meta);
        } else {
            he2_nh<WG>(G.g, h, hlen, lh, pre, voff, arena, arena + cap, cap);
            HE2_MARK(1);
            he2_compact<WG, BIG>(P, G, sh, arena, arena + cap, cap, nl_x, nl_meta);
        }
        HE2_MARK(2);
        const uint32_t K = sh.K;
        for (uint32_t i = tid; i < hlen; i += WG) hm[i] = G.g.h2v[sh.hoff + i];
        // --- vertices that two neighbours may share: a second row holding a vertex
        // finds its bit set and sets the bit in the second bitmap (the members are
        // stashed, so a row is gathered once)
        uint32_t* bm = BIG ? lds : arena + base0;
        if (!BIG) base0 += 2 * BM_WORDS;
        uint32_t* stash = arena + base0;
        const uint32_t room = base0 < AW ? AW - base0 : 0;  // words left for the stash and the survivors
        if (room) {
            for (uint32_t i = tid; i < 2 * BM_WORDS; i += WG) bm[i] = 0;
        }
        __syncthreads();
        if (room)
            he2_rows<WG>(G.g, sh, nl_x, nl_meta, row_at, K, nullptr, wpre, woff, true,
                         [&](uint32_t, uint32_t v, uint32_t j) {
                             if (j < room) stash[j] = v;
                             const uint32_t b = (v * 2654435761u) >> (32 - BM_LOG);
                             const uint32_t bit = 1u << (b & 31);
                             if (atomicOr(&bm[b >> 5], bit) & bit) atomicOr(&bm[BM_WORDS + (b >> 5)], bit);
                         });
        __syncthreads();
        const uint32_t W = sh.W;
        if (tid == 0) {
            // h's row and its members' incidence lists, each neighbour's row and metadata
            if (P.stats)
                atomicAdd((unsigned long long*)&st[1], (unsigned long long)(4ull * (hlen + lh) + 20ull * K + 4ull * W));
        }
        if (W > room || !room) {
            __syncthreads();
            move_on();
            continue;
        }
        // survivors (vertex, neighbour), from the arena's end downwards
        const uint32_t s_cap = (room - W) / 2;
        uint32_t* s_end = arena + AW;
        he2_rows<WG>(G.g, sh, nl_x, nl_meta, row_at, K, stash, wpre, woff, false,
                     [&](uint32_t xi, uint32_t v, uint32_t) {
                         const uint32_t b = (v * 2654435761u) >> (32 - BM_LOG);
                         if (!(bm[BM_WORDS + (b >> 5)] >> (b & 31) & 1u)) return;
                         const uint32_t q = atomicAdd(&sh.S, 1u);
                         if (q < s_cap) {
                             s_end[-1 - 2 * (int32_t)q] = xi;
                             s_end[-2 - 2 * (int32_t)q] = v;
                         }
                     });
        __syncthreads();
        const uint32_t S = sh.S;
        // --- exact groups: hash of the survivors' vertices, runs, and per neighbour its
        // shared vertices.  The regions go where they fit: over the bitmaps and the stash,
        // or over the hash of N(h).
        uint32_t lo_at = 0, hi_at = BIG ? base0 : base0 - 2 * BM_WORDS;
        const uint32_t lo_end = 2 * cap, hi_end = AW - 2 * S;
        bool fits = S <= s_cap;
        auto place = [&](uint32_t words) -> uint32_t {
            uint32_t r = 0;
            if (hi_at + words <= hi_end) { r = hi_at; hi_at += words; }
            else if (lo_at + words <= lo_end) { r = lo_at; lo_at += words; }
            else fits = false;
            return r;
        };
        const uint32_t vcap = hash_cap(S);
        uint32_t* tkey = arena + place(vcap);
        uint32_t* tcur = arena + place(vcap + 1);
        uint32_t* rx = arena + place(S);
        uint32_t* er = arena + place(S);
        uint32_t* ecur = arena + place(K);
        uint32_t* cnts = BIG ? lds : arena + place(NW * K > 2 * hlen + 2 ? NW * K : 2 * hlen + 2);
        if (!fits) {
            __syncthreads();
            move_on();
            continue;
        }
        for (uint32_t s = tid; s < vcap; s += WG) { tkey[s] = HGT_EMPTY; tcur[s] = 0; }
        for (uint32_t i = tid; i < K; i += WG) ecur[i] = 0;
        __syncthreads();
        for (uint32_t e = tid; e < S; e += WG) {
            uint32_t* pv = s_end - 2 - 2 * (int32_t)e;
            *pv = fr_add(tkey, tcur, vcap, *pv, 1u);
        }
        __syncthreads();
        HE2_MARK(4);
        // run starts (vertices of one neighbour only: an empty run), flagged when the vertex lies in h
        wg_prefix<WG>(vcap, sh.ws,
                      [&](uint32_t s) {
                          const uint32_t r = ld_at<BIG>(&tcur[s]) & POS;
                          return r >= 2 ? r : 0u;
                      },
                      [&](uint32_t s, uint32_t b) {
                          const uint32_t v = ld_at<BIG>(&tkey[s]);
                          const uint32_t in = v != HGT_EMPTY && contains_u32(hm, hlen, v) ? 1u : 0u;
                          tcur[s] = b | in << 31;
                      });
        if (tid == 0) {  // the end of the last run
            uint32_t t = 0;
            for (uint32_t w = 0; w < NW; w++) t += sh.ws[w];
            tcur[vcap] = t;
        }
        __syncthreads();
        for (uint32_t e = tid; e < S; e += WG) {
            uint32_t* pv = s_end - 2 - 2 * (int32_t)e;
            const uint32_t s = *pv;
            if ((ld_at<BIG>(&tcur[s + 1]) & POS) == (ld_at<BIG>(&tcur[s]) & POS)) *pv = HGT_EMPTY;
            else atomicAdd(&ecur[pv[1]], 1u);
        }
        __syncthreads();
        wg_prefix<WG>(K, sh.ws, [&](uint32_t i) { return ld_at<BIG>(&ecur[i]); },
                      [&](uint32_t i, uint32_t b) { ecur[i] = b; });
        __syncthreads();
        for (uint32_t e = tid; e < S; e += WG) {
            const uint32_t* pv = s_end - 2 - 2 * (int32_t)e;
            const uint32_t s = *pv;
            if (s == HGT_EMPTY) continue;
            const uint32_t xi = pv[1];
            rx[atomicAdd(&tcur[s], 1u) & POS] = xi;
            er[atomicAdd(&ecur[xi], 1u)] = s;
        }
        __syncthreads();
        // now run s is [end of s - 1, tcur[s]) and neighbour i's shared vertices [ecur[i-1], ecur[i])
        HE2_MARK(8);
        // --- disjoint-pair classes (the first slice); the histogram lies over the counters in the global stage
        if (slice == 0) {
            he2_disjoint<WG>(sh, T, A, nl_meta, K, hlen, cnts);
            __syncthreads();
        }
        HE2_MARK(3);
        // --- open paths h - x - y through the histograms, per eligible neighbour
        if (!P.static_mode)
            for (uint32_t i = tid; i < K; i += WG) {
                const uint32_t m = nl_meta[i], x = nl_x[i];
                if (meta_elig(m) && (nslice == 1 || slice_of(x, nslice) == slice)) he2_open(P, G, sh, A, x, m, st);
            }
        HE2_MARK(5);
        // --- intersecting neighbour pairs
        const uint32_t cw = BIG ? CNT_L : K;  // counters per wave
        uint32_t* cnt = cnts + wave * cw;
        for (uint32_t i = lane; i < cw; i += 64) cnt[i] = 0;
        wave_sync();
        // a wave's neighbours are every NW-th, looked at 64 at a time.  The slices of a centre
        // number its neighbours each in its own order, so a row belongs to the slice that its ID
        // names and a pair to its row of smaller ID; unsliced, a pair belongs to its earlier row.
        for (uint32_t c0 = 0; c0 * NW < K; c0 += 64) {
          const uint32_t il = wave + NW * (c0 + lane);
          uint32_t mx_l = 0, e0_l = 0, e1_l = 0, x_l = 0;
          if (il < K) {
              mx_l = nl_meta[il];
              e0_l = il ? ld_at<BIG>(&ecur[il - 1]) : 0;
              e1_l = ld_at<BIG>(&ecur[il]);
              if (nslice > 1) x_l = nl_x[il];
          }
          uint64_t rows = __ballot(il < K && meta_elig(mx_l) && e0_l < e1_l &&
                                   (nslice == 1 || slice_of(x_l, nslice) == slice));
          for (; rows; rows &= rows - 1) {
            const int r = __ffsll((unsigned long long)rows) - 1;
            const uint32_t i = wave + NW * (c0 + r);
            const uint32_t mx = __shfl(mx_l, r, 64), e0 = __shfl(e0_l, r, 64), e1 = __shfl(e1_l, r, 64);
            const uint32_t x = __shfl(x_l, r, 64);
            // lanes in groups, a group per shared vertex: few vertices, wide groups
            const uint32_t ne = e1 - e0;
            const uint32_t glog = ne == 1 ? 6 : ne == 2 ? 5 : ne <= 8 ? 4 : ne <= 16 ? 3 : 2;
            const uint32_t ng = 64u >> glog, gid = lane >> glog, sub = lane & ((1u << glog) - 1);
            auto walk = [&](uint32_t w0, uint32_t w1, auto fn) {
                for (uint32_t e = e0 + gid; e < e1; e += ng) {
                    const uint32_t s = er[e];
                    const uint32_t r0 = s ? ld_at<BIG>(&tcur[s - 1]) & POS : 0, t1 = ld_at<BIG>(&tcur[s]);
                    for (uint32_t j = r0 + sub; j < (t1 & POS); j += 1u << glog) {
                        const uint32_t y = rx[j];
                        if (y >= w0 && y < w1) fn(y, t1 >> 31);
                    }
                }
            };
            for (uint32_t w0 = nslice == 1 ? i + 1 : 0; w0 < K; w0 += cw) {
                const uint32_t w1 = K - w0 < cw ? K : w0 + cw;
                walk(w0, w1, [&](uint32_t y, uint32_t in) { atomicAdd(&cnt[y - w0], 1u + (in << 16)); });
                wave_sync();
                walk(w0, w1, [&](uint32_t y, uint32_t) {
                    const uint32_t v = atomicExch(&cnt[y - w0], 0u);
                    if (!v || (nslice > 1 && nl_x[y] <= x)) return;  // taken at another shared vertex, or row
                    const uint32_t my = nl_meta[y];
                    if (meta_elig(my)) he2_pair(P, T, A, hlen, mx, my, v & 0xffffu, v >> 16);
                });
                wave_sync();
                folded += w1 - w0;
            }
            if (folded >= FOLD_AT) {
                pair_fold(A);
                folded = 0;
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
__device__ void he2_flush_stats(const He2Params& P, const uint64_t* st, const uint64_t* ph) {
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

template <bool BIG, int WG>
__device__ __forceinline__ void he2_kernel(const He2Params& P, uint32_t* arena, uint32_t words, uint32_t* lds) {
    __shared__ Sh2 sh;
    __shared__ Tables T;
    __shared__ He2Acc A;
    __shared__ uint64_t st[2];
    __shared__ uint64_t ph[HE2_PHASES];
    const uint32_t tid = threadIdx.x;
    if (tid < HE2_PHASES) ph[tid] = 0;
    if (tid == 0) sh.cur_g = 0xffffffffu;
    for (uint32_t i = tid; i < 128; i += WG) T.he[i] = P.he_tab[i];
    for (uint32_t i = tid; i < HGT_N_HE_CLASSES * COPIES; i += WG) A.pair[i] = 0;
    for (uint32_t i = tid; i < 8 * COPIES; i += WG) A.open[i] = 0;
    if (tid < HGT_N_HE_CLASSES) A.tot[tid] = 0;
    // open path: h & x (8) and x & y (16), h only (1), x only (2), y only (4)
    if (tid < 8) A.cls8[tid] = P.he_tab[24 | (tid & 4 ? 1 : 0) | (tid & 2 ? 2 : 0) | (tid & 1 ? 4 : 0)];
    if (tid < 2) st[tid] = 0;
    __syncthreads();
    he2_body<BIG, WG>(P, arena, words, lds, sh, T, A, st, ph);
    he2_flush_graph<WG>(P, sh.cur_g, A);
    he2_flush_stats<BIG ? 2 : 0>(P, st, ph);
}

__global__ void __launch_bounds__(HGT_WG) k_he2_s0(He2Params P) {
    __shared__ __attribute__((aligned(16))) uint32_t arena[ARENA_S];
    he2_kernel<false, HGT_WG>(P, arena, ARENA_S, nullptr);
}

__global__ void __launch_bounds__(WG_L, 4) k_he2_s2(He2Params P) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[LDS_L];
    he2_kernel<true, WG_L>(P, P.garena + (uint64_t)blockIdx.x * P.garena_words, (uint32_t)P.garena_words, lds);
}

// Slices of the global stage's centres, one wave per centre: the pairs along its
// members' lists (sum of the squared list lengths) over SLICE_PAIRS.  A launch of few
// centres cuts finer, so that one dense centre does not outlast the rest.
constexpr uint64_t SLICE_PAIRS = 1ull << 19;
constexpr uint32_t SLICES_MAX = 64;
__global__ void k_he2_slices(Multi M, const uint64_t* __restrict__ list, const uint32_t* n_p, uint64_t cap,
                             uint32_t slice_lh, uint64_t slice_pairs, uint64_t* pre) {
    const int lane = threadIdx.x & 63;
    const uint64_t c = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t n = *n_p;
    if (c == 0 && lane == 0) pre[cap] = n;
    if (c >= n) return;
    const uint64_t it = list[c];
    const GraphView& g = M.graphs[(uint32_t)(it >> 32)].g;
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
    if (lane == 0) {
        const uint64_t full = slice_pairs ? slice_pairs : SLICE_PAIRS;
        const uint64_t per = n >= 512 ? full : (full * n / 512 > full / 16 ? full * n / 512 : full / 16);
        uint64_t sl = slice_lh ? (lh + slice_lh - 1) / slice_lh : (sq + per - 1) / per;
        pre[c] = sl < 1 ? 1 : (sl > SLICES_MAX ? SLICES_MAX : sl);
    }
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
    k_bl_count<<<g, 256, 0, s>>>(P.n_entries, P.entries_cap, P.ent_x, bl_cnt);
    hgt_scan_u64(bl_cnt, bl_off, n_ids, nullptr, nullptr, scan_tmp, s);
    (void)hipMemcpyAsync(bl_cur, bl_off, n_ids * 8, hipMemcpyDeviceToDevice, s);
    k_bl_scatter<<<g, 256, 0, s>>>(P.n_entries, P.entries_cap, P.ent_x, P.ent_d, P.ent_pay, bl_cur, bl_d, bl_pay);
}

void he2_remove_deleted(NbrParams& P, hipStream_t s) {
    if (P.M.total == 0) return;
    k_h_remove<<<2048, 256, 0, s>>>(P.M, P.n_entries, P.entries_cap, P.ent_x, P.ent_pay);
}

void he2_launch_lds(He2Params& P, unsigned grid, hipStream_t s) {
    if (P.M.total) k_he2_s0<<<grid, HGT_WG, 0, s>>>(P);
}

void he2_launch_global(He2Params& P, unsigned grid, hipStream_t s) {
    if (!P.M.total) return;
    const uint64_t cap = P.slice_cap;
    k_he2_slices<<<(unsigned)((cap * 64 + 255) / 256), 256, 0, s>>>(P.M, P.list[0], &P.count[0], cap, P.slice_lh,
                                                                    P.slice_pairs, P.slice_pre);
    hgt_scan_u64(P.slice_pre, P.slice_pre, cap, P.slice_pre + cap, P.slice_pre + cap + 1, P.slice_scan_tmp, s);
    k_he2_s2<<<grid, WG_L, 0, s>>>(P);
}
