// triad_iv.hip -- incident-vertex triad deltas (types 1-3 with hyperedge multiplicity).
//
// With m_p the number of hyperedges containing the vertex pair p and
// w_p = sum over those hyperedges of (|h| - 2):
//   type 1            = sum_h C(|h|,3)
//   type 1+2+3        = sum over vertex triangles {a,b,c} of m_ab m_bc m_ac
//   type 2            = sum_p m_p w_p - 3 * type 1
// (a type-2 tuple is a vertex triple inside one hyperedge with one of its
// three pairs re-witnessed by a different hyperedge).  Only pairs inside a
// changed hyperedge ("touched" pairs) change m_p, so a batch changes
//   sum_p m_p w_p             by its value over the touched pairs, and
//   the triangle sum          by its value over triangles with a touched pair.
// Both are evaluated on the old graph (before the batch) and on the new graph
// (after it); the difference is the delta.
//
// Every touched pair has an owner, its endpoint of higher degree.  A wave (small
// owners) or a workgroup takes an owner a and builds its clique map M_a : w -> m_aw
// from the hyperedges that contain a, in LDS.  For each touched pair (a, b) it owns,
// m_ab is read from the map, w_ab is met in the scan of b's hyperedges, and the
// triangles through (a, b) contribute
//   m_ab * sum_{h' containing b} sum_{w in h', w != a, b} M_a[w]
// (the inner double sum counts w with multiplicity m_bw; b, the endpoint of
// lower degree, is the one scanned).  A triangle with several touched pairs is
// counted at its lexicographically smallest one: the triangle {a, b, w} is skipped
// when {a, w} is touched and w < b, or {b, w} is touched and w < a (a global hash of
// the touched pairs answers).
//
// What bounds it: chains of dependent gathers (pair, b's list, row length and offset,
// members, the map, the touched hash).  So the hyperedges of up to 64 pairs are laid
// end to end and taken 64 at a time, their members laid end to end again: one chain
// serves about 64 hyperedges instead of one pair's twenty, no lane waits for a longer
// row, and the sums need no reduction per pair.  Members that may be in the map are
// queued in LDS and the touched hash is asked for 128 of them at once, instead of
// stalling each step of the scan.  Owners are cut every 64 pairs, so none outlasts the
// rest, and taken and moved on several at a time (an atomic of one address passes every
// 13 ns: one per owner bound the whole kernel).
#include "triad_common.h"

namespace {

using namespace tri;

constexpr uint32_t IV_ARENA = 5888;       // stage 1: 23 KB of LDS per workgroup
constexpr uint32_t IV_WAVE_WORDS = 1024;  // stage 0: 4 KB of LDS per wave

__device__ __forceinline__ uint64_t pair_key(uint32_t x, uint32_t y) {
    return x < y ? ((uint64_t)x << 32 | y) : ((uint64_t)y << 32 | x);
}

// The rest of touched() once the first slot t is read.
__device__ __forceinline__ bool touched_from(const uint64_t* tab, uint64_t mask, uint64_t k, uint64_t t) {
    uint64_t s = mix64(k) & mask;
    for (uint64_t probe = 0; probe <= mask; probe++) {
        if (t == k) return true;
        if (t == ~0ull) return false;
        s = (s + 1) & mask;
        t = tab[s];
    }
    return false;
}

__device__ __forceinline__ bool touched(const uint64_t* tab, uint64_t mask, uint32_t x, uint32_t y) {
    const uint64_t k = pair_key(x, y);
    return touched_from(tab, mask, k, tab[mix64(k) & mask]);
}

__global__ void k_iv_hash_build(const uint64_t* __restrict__ pairs, const uint64_t* n_p, uint64_t* tab, uint64_t mask) {
    uint64_t n = *n_p;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t k = pairs[i];
        uint64_t s = mix64(k) & mask;
        for (uint64_t probe = 0; probe <= mask; probe++) {
            unsigned long long prev = atomicCAS((unsigned long long*)&tab[s], ~0ull, (unsigned long long)k);
            if (prev == ~0ull || prev == k) break;
            s = (s + 1) & mask;
        }
    }
}

__global__ void k_iv_owner_heads(const uint64_t* __restrict__ pairs, const uint64_t* n_p, uint64_t* head) {
    uint64_t n = *n_p;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        head[i] = iv_head(pairs, i) ? 1 : 0;
}

__global__ void k_iv_owner_list(const uint64_t* __restrict__ pairs, const uint64_t* n_p, const uint64_t* __restrict__ pos,
                                uint64_t* owner_start, const uint64_t* n_owner) {
    uint64_t n = *n_p;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        if (iv_head(pairs, i)) owner_start[pos[i]] = i;
    if (blockIdx.x == 0 && threadIdx.x == 0) owner_start[*n_owner] = n;
}

// ---- memory-free fallback for vertices whose map does not fit: per pair,
// m_ab from binary searches and every triangle vertex c from a's hyperedges
// (taken at the first of them that holds c), m_ac and m_bc by list intersection.
// |A & B| for two incidence lists and their first common element in list order
// (both lists are sorted by the same key, so it is the same in either list)
__device__ __forceinline__ uint32_t inter_count_min(const GraphView& g, const uint32_t* A, uint32_t na,
                                                    const uint32_t* B, uint32_t nb, uint32_t* mn) {
    if (na > nb) {
        const uint32_t* t = A; A = B; B = t;
        uint32_t n = na; na = nb; nb = n;
    }
    uint32_t c = 0, first = HGT_EMPTY;
    for (uint32_t i = 0; i < na; i++) {
        uint32_t e = A[i];
        if (v2h_contains(g, B, nb, e)) {
            if (c == 0) first = e;
            c++;
        }
    }
    *mn = first;
    return c;
}

// one wave: returns (lane 0) m_ab * w_ab in *s_out and the attributed triangle sum in *t_out
__device__ void iv_pair_direct(const IvJob& P, uint32_t a, uint32_t b, uint32_t* pre, uint64_t* s_out,
                               uint64_t* t_out) {
    const int lane = threadIdx.x & 63;
    uint32_t la = P.g.v_len[a], lb = P.g.v_len[b];
    if (lb < la) { uint32_t t = a; a = b; b = t; t = la; la = lb; lb = t; }
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    const uint32_t* A = P.g.v2h + P.g.v_off[a];
    const uint32_t* B = P.g.v2h + P.g.v_off[b];
    uint64_t m = 0, w = 0;
    for (uint32_t i = lane; i < la; i += 64) {
        uint32_t h = A[i];
        uint32_t d = P.g.h_len[h];
        if (contains_u32(P.g.h2v + P.g.h_off[h], d, b)) { m++; w += d - 2; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        m += __shfl_xor(m, o, 64);
        w += __shfl_xor(w, o, 64);
    }
    *s_out = m * w;
    uint64_t t_sum = 0;
    if (m) {
        for (uint32_t base = 0; base < la; base += 64) {
            uint32_t cnt = la - base < 64 ? la - base : 64;
            uint32_t d = 0;
            if ((uint32_t)lane < cnt) d = P.g.h_len[A[base + lane]];
            uint32_t inc = d;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                uint32_t t = __shfl_up(inc, o, 64);
                if (lane >= o) inc += t;
            }
            if ((uint32_t)lane < cnt) pre[lane + 1] = inc;
            if (lane == 0) pre[0] = 0;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            uint32_t tot = pre[cnt];
            for (uint32_t p = lane; p < tot; p += 64) {
                uint32_t k = seg_of<uint32_t>(pre, cnt, p);
                uint32_t hk = A[base + k];
                uint32_t c = P.g.h2v[P.g.h_off[hk] + (p - pre[k])];
                if (c == a || c == b) continue;
                const uint32_t* C = P.g.v2h + P.g.v_off[c];
                uint32_t lc = P.g.v_len[c];
                uint32_t first;
                uint32_t mac = inter_count_min(P.g, A, la, C, lc, &first);
                if (first != hk) continue;
                uint32_t dummy;
                uint32_t mbc = inter_count_min(P.g, B, lb, C, lc, &dummy);
                if (mbc == 0) continue;
                if (c < hi && touched(P.tab, P.tab_mask, lo, c)) continue;
                if (c < lo && touched(P.tab, P.tab_mask, hi, c)) continue;
                t_sum += m * (uint64_t)mac * (uint64_t)mbc;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t_sum += __shfl_xor(t_sum, o, 64);
    *t_out = t_sum;
}

// The clique map of an owner a: m_aw by w, open addressing over cap slots, keys and
// counts apart so that the probes of a wave read consecutive key words; 2 words per
// slot.  (w_ab is needed for the owned pairs only, whose scan of b meets a itself.)
struct IvMap {
    uint32_t* key;
    uint32_t* m;
    uint32_t cap;
};

template <bool GLOBAL>
__device__ __forceinline__ uint32_t ld_map(const uint32_t* p) {  // written by atomics: global words are read in the L2
    if (GLOBAL) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}

// The sieve in front of the map: most members of b's hyperedges are not in M_a, and one
// bit tells so for all but a few of them (8192 bits: an owner of 1,000 keys lets 12% by).
constexpr uint32_t IV_SIEVE = 256;  // words
__device__ __forceinline__ uint32_t iv_bit(uint32_t w) { return (w * 0x9e3779b1u) >> 19; }

// m_aw, 0 when w is not in the map (a count is never 0)
template <bool GLOBAL>
__device__ __forceinline__ uint32_t map_find(const IvMap& mp, uint32_t key) {
    const uint32_t cap = mp.cap;
    uint32_t s = (uint32_t)(((uint64_t)(key * 2654435761u) * cap) >> 32);
    for (uint32_t probe = 0; probe < cap; probe++) {
        const uint32_t k = ld_map<GLOBAL>(&mp.key[s]);
        if (k == key) return ld_map<GLOBAL>(&mp.m[s]);
        if (k == HGT_EMPTY) return 0;
        s = s + 1 == cap ? 0 : s + 1;
    }
    return 0;
}

__device__ __forceinline__ void map_add(const IvMap& mp, uint32_t key) {
    const uint32_t cap = mp.cap;
    uint32_t s = (uint32_t)(((uint64_t)(key * 2654435761u) * cap) >> 32);
    for (uint32_t probe = 0; probe < cap; probe++) {
        uint32_t k = __atomic_load_n(&mp.key[s], __ATOMIC_RELAXED);
        if (k == HGT_EMPTY) {
            uint32_t prev = atomicCAS(&mp.key[s], HGT_EMPTY, key);
            if (prev == HGT_EMPTY || prev == key) break;
        } else if (k == key) {
            break;
        }
        s = s + 1 == cap ? 0 : s + 1;
    }
    atomicAdd(&mp.m[s], 1u);
}

// Up to 64 pairs of an owner, their hyperedges laid end to end.
struct IvTile {
    uint32_t b[64], m[64], pre[65];
    uint64_t off[64];
};
// A wave's own: the rows of 64 of those hyperedges, and the members that may be in the
// map and are not classified yet.
struct IvWave {
    Flat f;
    uint32_t len[64], pk[64];
    uint64_t off[64];
    uint32_t qw[192], qk[192];
};
struct IvSh {
    uint32_t oi, stop;
    uint32_t ws[NWAVE];
};

// One owner by NW waves (1: each wave alone, 4: the workgroup together).  Returns false,
// with nothing counted, when the map does not fit the arena.
template <int NW, bool GLOBAL>
__device__ bool iv_owner(const IvJob& P, uint32_t oi, uint32_t* arena, uint32_t arena_words, bool pass_on, uint32_t* sieve,
                         IvTile& tile, IvWave& W, uint32_t* ws, uint64_t& s_sum, uint64_t& t_sum, uint64_t& bytes) {
    const uint32_t lane = threadIdx.x & 63, wave = NW == 1 ? 0 : threadIdx.x >> 6;
    const uint32_t tid = NW == 1 ? lane : threadIdx.x;
    auto sync = [] {
        if (NW == 1) wave_sync();
        else __syncthreads();
    };
    const uint64_t p0 = P.owner_start[oi], p1 = P.owner_start[oi + 1];
    const uint32_t a = (uint32_t)(P.pairs[p0] >> 32);
    const uint32_t la = P.g.v_len[a];
    const uint32_t* A = P.g.v2h + P.g.v_off[a];
    // L = sum of the cardinalities of a's hyperedges, up to 64 a wave at a time (few: shared
    // among the waves); the first rows' lengths and offsets are kept for the map
    const uint32_t per = la / NW + 1 < 64 ? la / NW + 1 : 64;
    uint32_t L = 0, d0 = 0;
    uint64_t off0 = 0;
    for (uint32_t i = wave * per; i < la; i += NW * per)
        if (lane < per && i + lane < la) {
            const uint32_t h = A[i + lane], d = P.g.h_len[h];
            L += d;
            if (i == wave * per) {
                d0 = d;
                off0 = P.g.h_off[h];
            }
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) L += __shfl_xor(L, o, 64);
    if (NW > 1) {
        if (lane == 0) ws[wave] = L;
        __syncthreads();
        L = 0;
        for (int w = 0; w < NW; w++) L += ws[w];
    }
    const uint64_t need = (uint64_t)L + L / 2 + 32;
    if (pass_on || 2 * need > arena_words) return false;
    const uint32_t cap = (uint32_t)need;
    const IvMap mp{arena, arena + cap, cap};
    for (uint32_t s = tid; s < cap; s += NW * 64) {
        mp.key[s] = HGT_EMPTY;
        mp.m[s] = 0;
    }
    for (uint32_t s = tid; s < IV_SIEVE; s += NW * 64) sieve[s] = 0;
    sync();
    // M_a from a's hyperedges and the sieve, a bitmap of its keys
    for (uint32_t i = wave * per; i < la; i += NW * per) {
        const uint32_t n = la - i < per ? la - i : per;
        uint32_t d = d0;
        W.off[lane] = off0;
        if (i != wave * per) {
            d = 0;
            if (lane < n) {
                const uint32_t h = A[i + lane];
                d = P.g.h_len[h];
                W.off[lane] = P.g.h_off[h];
            }
        }
        wave_flat<4>(W.f, d, [&](uint32_t l, uint32_t r) { return P.g.h2v[W.off[l] + r]; },
                     [&](bool ok, uint32_t, uint32_t, uint32_t, uint32_t w) {
                         if (!ok || w == a) return;
                         const uint32_t b = iv_bit(w);
                         atomicOr(&sieve[b >> 5], 1u << (b & 31));
                         map_add(mp, w);
                     });
    }
    if (lane == 0 && P.stats) bytes += 4ull * (la + L) / NW;
    sync();
    uint32_t qn = 0;  // queued members, wave-uniform
    // two members a lane at a time, their first probes of the touched hash all in flight together
    auto classify = [&](uint32_t from, uint32_t n) {
        uint32_t m[2] = {0, 0}, b[2], w[2];
        uint64_t wt[2], k1[2], k2[2], t1[2], t2[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const uint32_t i = 64 * u + lane;
            t1[u] = t2[u] = ~0ull;
            b[u] = w[u] = 0;
            wt[u] = k1[u] = k2[u] = 0;
            if (i >= n) continue;
            w[u] = W.qw[from + i];
            const uint32_t k = W.qk[from + i];
            m[u] = map_find<GLOBAL>(mp, w[u]);
            if (!m[u]) continue;
            b[u] = tile.b[k];
            wt[u] = (uint64_t)tile.m[k] * m[u];
            k1[u] = pair_key(a, w[u]);
            k2[u] = pair_key(b[u], w[u]);
            if (w[u] < b[u]) t1[u] = P.tab[mix64(k1[u]) & P.tab_mask];
            if (w[u] < a) t2[u] = P.tab[mix64(k2[u]) & P.tab_mask];
        }
#pragma unroll
        for (int u = 0; u < 2; u++)
            if (m[u] && !touched_from(P.tab, P.tab_mask, k1[u], t1[u]) && !touched_from(P.tab, P.tab_mask, k2[u], t2[u]))
                t_sum += wt[u];
    };
    for (uint64_t q0 = p0; q0 < p1; q0 += 64) {
        const uint32_t np = p1 - q0 < 64 ? (uint32_t)(p1 - q0) : 64;
        if (wave == 0) {
            uint32_t lb = 0;
            if (lane < np) {
                const uint32_t b = (uint32_t)P.pairs[q0 + lane];
                const uint32_t m = map_find<GLOBAL>(mp, b);
                tile.b[lane] = b;
                tile.m[lane] = m;
                tile.off[lane] = P.g.v_off[b];
                lb = m ? P.g.v_len[b] : 0;  // m_ab = 0: nothing to count
            }
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(lb, o, 64);
                if (lane >= (uint32_t)o) lb += t;
            }
            tile.pre[lane + 1] = lb;
            if (lane == 0) tile.pre[0] = 0;
        }
        sync();
        const uint32_t items = tile.pre[np];
        const uint32_t step = NW == 1 || items >= NW * 64 ? 64 : items / NW + 1;
        for (uint32_t c = wave * step; c < items; c += NW * step) {
            const uint32_t n = items - c < step ? items - c : step;
            uint32_t d = 0;
            if (lane < n) {
                const uint32_t k = seg_of<uint32_t>(tile.pre, np, c + lane);
                const uint32_t h = P.g.v2h[tile.off[k] + (c + lane - tile.pre[k])];
                d = P.g.h_len[h];
                W.off[lane] = P.g.h_off[h];
                W.len[lane] = d;
                W.pk[lane] = k;
            }
            const uint32_t tot = wave_flat<4>(W.f, d, [&](uint32_t l, uint32_t r) { return P.g.h2v[W.off[l] + r]; },
                [&](bool ok, uint32_t l, uint32_t, uint32_t, uint32_t w) {
                    const uint32_t k = W.pk[l];
                    bool may = false;
                    if (ok) {
                        const uint32_t b = iv_bit(w);
                        may = sieve[b >> 5] >> (b & 31) & 1u;
                        if (w == a) {
                            s_sum += (uint64_t)tile.m[k] * (W.len[l] - 2);
                            may = false;
                        }
                        if (may && w == tile.b[k]) may = false;
                    }
                    const uint64_t hit = __ballot(may);
                    if (!hit) return;
                    if (may) {
                        const uint32_t q = qn + __popcll(hit & ((1ull << lane) - 1));
                        W.qw[q] = w;
                        W.qk[q] = k;
                    }
                    qn += __popcll(hit);
                    if (qn >= 128) {
                        wave_sync();
                        qn -= 128;
                        classify(qn, 128);
                        wave_sync();
                    }
                });
            if (P.stats && lane == 0) bytes += 4ull * (n + tot);
        }
        wave_sync();
        classify(0, qn);
        qn = 0;
        sync();
    }
    return true;
}

__device__ __forceinline__ void iv_add(const IvJob& P, uint64_t s_sum, uint64_t t_sum, uint64_t bytes) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s_sum += __shfl_xor(s_sum, o, 64);
        t_sum += __shfl_xor(t_sum, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (s_sum) atomicAdd((unsigned long long*)&P.out[0], (unsigned long long)s_sum);
        if (t_sum) atomicAdd((unsigned long long*)&P.out[1], (unsigned long long)t_sum);
        if (bytes && P.stats) atomicAdd((unsigned long long*)&P.stats[ST_IV_BYTES], (unsigned long long)bytes);
    }
}

// The graphs of a launch in turn, each workgroup from a graph of its own: one graph's
// owners end with a few long ones, which leave most of the chip idle (a served round of 16
// graphs: 21.9 ms with one launch per graph and stage, 15.4 ms with one per stage).
__device__ __forceinline__ uint32_t iv_turn(uint32_t k, uint32_t n) {
    return (k + (uint32_t)((uint64_t)blockIdx.x * n / gridDim.x)) % n;
}
__device__ __forceinline__ uint32_t iv_taken(const uint32_t* queue) {  // a look before the atomic
    return __hip_atomic_load(queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Stage 0: every wave takes owners of its own; maps of up to IV_WAVE_WORDS / 2 slots.
// Three quarters of the owners of a power-law graph fit, and 16 of them share a CU (four
// workgroups of four waves, 40 KB of LDS each) where workgroup-sized ones leave it to four.
__global__ void __launch_bounds__(HGT_WG) k_iv_wave(IvParams A) {
    __shared__ __attribute__((aligned(16))) uint32_t arena[NWAVE][IV_WAVE_WORDS];
    __shared__ uint32_t sieve[NWAVE][IV_SIEVE];
    __shared__ IvTile tile[NWAVE];
    __shared__ IvWave W[NWAVE];
    __shared__ uint32_t moved[NWAVE][32];  // owners this wave moves on, appended 32 at a time
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t k = 0; k < A.n_jobs; k++) {
        const IvJob& P = A.job[iv_turn(k, A.n_jobs)];
        if (*((volatile const int32_t*)P.status)) continue;  // no barrier below
        const uint64_t n = *P.n_owners;
        if (k && iv_taken(&P.queue[0]) >= n) continue;
        uint64_t s_sum = 0, t_sum = 0, bytes = 0;
        const uint32_t take = take_size(n, gridDim.x * NWAVE, 2);
        uint32_t q = 0, n_moved = 0;
        auto append = [&]() {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&P.queue[4], n_moved);
            at = __shfl(at, 0, 64);
            wave_sync();
            if (lane < n_moved) A.list[0][P.list_at + at + lane] = moved[wave][lane];
            wave_sync();
            n_moved = 0;
        };
        if (lane == 0) q = atomicAdd(&P.queue[0], take);
        for (;;) {
            const uint32_t first = __shfl(q, 0, 64);
            if (first >= n) break;
            if (lane == 0) q = atomicAdd(&P.queue[0], take);  // the next ones, while these run
            const uint32_t last = n - first < take ? (uint32_t)n : first + take;
            for (uint32_t oi = first; oi < last; oi++) {
                if (!iv_owner<1, false>(P, oi, arena[wave], IV_WAVE_WORDS, P.force_direct || 0 < P.force_stage,
                                        sieve[wave], tile[wave], W[wave], nullptr, s_sum, t_sum, bytes)) {
                    if (lane == 0) moved[wave][n_moved] = oi;
                    if (++n_moved == 32) append();
                }
                wave_sync();
            }
        }
        if (n_moved) append();
        iv_add(P, s_sum, t_sum, bytes);
    }
}

// Stages 1 (23 KB of LDS), 2 and 3 (global arenas): a workgroup per owner.
template <int STAGE>
__device__ void iv_body(const IvParams& A, uint32_t* arena, uint32_t arena_words) {
    __shared__ IvSh sh;
    __shared__ uint32_t sieve[IV_SIEVE];
    __shared__ IvTile tile;
    __shared__ IvWave W[NWAVE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (uint32_t k = 0; k < A.n_jobs; k++) {
        const IvJob& P = A.job[iv_turn(k, A.n_jobs)];
        uint32_t n = 0;
        if (tid == 0) {  // read once per workgroup: every thread takes the same way past the barriers below
            n = *((volatile const int32_t*)P.status) ? 0u : P.queue[3 + STAGE];
            sh.stop = n == 0 || (k && iv_taken(&P.queue[STAGE]) >= n);
        }
        __syncthreads();
        const uint32_t none = sh.stop;
        __syncthreads();
        if (none) continue;
        uint64_t s_sum = 0, t_sum = 0, bytes = 0;
        const uint32_t take = take_size(n, gridDim.x);
        uint32_t q = 0, q_end = 0;
        for (;;) {
            if (tid == 0) {
                if (q == q_end) {
                    q = atomicAdd(&P.queue[STAGE], take);
                    q_end = q + take;
                }
                sh.stop = q >= n;
                if (!sh.stop) sh.oi = A.list[STAGE - 1][P.list_at + q++];
            }
            __syncthreads();
            if (sh.stop) break;
            const uint32_t oi = sh.oi;
            // the tests' stage numbers: the first two stages are one to them
            const bool pass_on = P.force_direct || STAGE - 1 < P.force_stage;
            if (!iv_owner<NWAVE, STAGE != 1>(P, oi, arena, arena_words, pass_on, sieve, tile, W[wave], sh.ws,
                                             s_sum, t_sum, bytes)) {
                if (STAGE < 3) {
                    if (tid == 0) A.list[STAGE][P.list_at + atomicAdd(&P.queue[4 + STAGE], 1u)] = oi;
                } else {  // too large for any map: pair by pair without one
                    const uint64_t p0 = P.owner_start[oi], p1 = P.owner_start[oi + 1];
                    const uint32_t a = (uint32_t)(P.pairs[p0] >> 32);
                    for (uint64_t q = p0 + wave; q < p1; q += NWAVE) {
                        uint64_t so, to;
                        iv_pair_direct(P, a, (uint32_t)P.pairs[q], W[wave].f.bits, &so, &to);
                        if (lane == 0) {
                            s_sum += so;
                            t_sum += to;
                        }
                    }
                }
            }
            __syncthreads();
        }
        __syncthreads();  // sh.stop has been read by all
        iv_add(P, s_sum, t_sum, bytes);
    }
}

__global__ void __launch_bounds__(HGT_WG) k_iv_lds(IvParams A) {
    __shared__ __attribute__((aligned(16))) uint32_t arena[IV_ARENA];
    iv_body<1>(A, arena, IV_ARENA);
}

template <int STAGE>
__global__ void __launch_bounds__(HGT_WG) k_iv_global(IvParams A) {
    uint32_t* arena = STAGE == 2 ? A.garena + (uint64_t)blockIdx.x * A.garena_words
                                 : A.garena2 + (uint64_t)blockIdx.x * A.garena2_words;
    iv_body<STAGE>(A, arena, (uint32_t)(STAGE == 2 ? A.garena_words : A.garena2_words));
}

__global__ void k_iv_begin(IvParams A) {
    const uint32_t j = threadIdx.x >> 3, w = threadIdx.x & 7;
    if (j < A.n_jobs && w < 7) A.job[j].queue[w] = 0;
}

}  // namespace

void iv_touched_build(const uint64_t* canon, const uint64_t* own, const uint64_t* n_pairs, uint64_t* tab,
                      uint64_t tab_slots, uint64_t* head, uint64_t* owner_start, uint64_t* n_owners, uint64_t pairs_cap,
                      void* scan_tmp, hipStream_t s) {
    hgt_fill_u64(tab, ~0ull, tab_slots, s);
    k_iv_hash_build<<<2048, 256, 0, s>>>(canon, n_pairs, tab, tab_slots - 1);
    k_iv_owner_heads<<<2048, 256, 0, s>>>(own, n_pairs, head);
    hgt_scan_u64(head, head, pairs_cap, n_pairs, n_owners, scan_tmp, s);
    k_iv_owner_list<<<2048, 256, 0, s>>>(own, n_pairs, head, owner_start, n_owners);
}

void triad_iv_launch(const IvParams& P, unsigned grid_wave, unsigned grid_lds, unsigned grid_global,
                     unsigned grid_global2, hipStream_t s) {
    static_assert(sizeof(IvParams) <= 4096, "kernel arguments");
    k_iv_begin<<<1, 8 * kIvJobs, 0, s>>>(P);
    k_iv_wave<<<grid_wave, HGT_WG, 0, s>>>(P);
    k_iv_lds<<<grid_lds, HGT_WG, 0, s>>>(P);
    k_iv_global<2><<<grid_global, HGT_WG, 0, s>>>(P);
    k_iv_global<3><<<grid_global2, HGT_WG, 0, s>>>(P);
}
