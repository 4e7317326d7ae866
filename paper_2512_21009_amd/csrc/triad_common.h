// triad_common.h -- device helpers shared by the triad-delta kernels.
#pragma once

#include "triad.h"

namespace tri {

constexpr int NWAVE = HGT_WG / HGT_WAVE;  // 4

// meta word of a neighbour: c (14 bits) | len << 14 | eligible << 28 | in window << 29
__device__ __forceinline__ uint32_t meta_c(uint32_t m) { return m & 0x3fffu; }
__device__ __forceinline__ uint32_t meta_len(uint32_t m) { return (m >> 14) & 0x3fffu; }
__device__ __forceinline__ bool meta_elig(uint32_t m) { return (m >> 28) & 1u; }
__device__ __forceinline__ bool meta_win(uint32_t m) { return (m >> 29) & 1u; }

__device__ __forceinline__ int venn_code(int na, int nb, int nc, int ab, int bc, int ca, int abc) {
    int c = 0;
    c |= (na - ab - ca + abc > 0) ? 1 : 0;
    c |= (nb - ab - bc + abc > 0) ? 2 : 0;
    c |= (nc - bc - ca + abc > 0) ? 4 : 0;
    c |= (ab - abc > 0) ? 8 : 0;
    c |= (bc - abc > 0) ? 16 : 0;
    c |= (ca - abc > 0) ? 32 : 0;
    c |= (abc > 0) ? 64 : 0;
    return c;
}

__device__ __forceinline__ bool key_before(int64_t ta, uint64_t sa, int64_t tb, uint64_t sb) {
    return ta < tb || (ta == tb && sa < sb);
}

// Venn code of the triple (h, x, y) relabelled in arrival order.
__device__ __forceinline__ int time_code(int64_t th, uint64_t sh, int64_t tx, uint64_t sx, int64_t ty, uint64_t sy,
                                         int nh, int nx, int ny, int hx, int xy, int hy, int hxy) {
    // rank of each label in arrival order
    int rh = (int)key_before(tx, sx, th, sh) + (int)key_before(ty, sy, th, sh);
    int rx = (int)key_before(th, sh, tx, sx) + (int)key_before(ty, sy, tx, sx);
    int lab[3];
    lab[rh] = 0;
    lab[rx] = 1;
    lab[3 - rh - rx] = 2;
    int n[3] = {nh, nx, ny};
    // pairwise intersections indexed by label pair
    auto pr = [&](int a, int b) -> int {
        int s = a + b;  // {0,1}->1 hx, {1,2}->3 xy, {0,2}->2 hy
        return s == 1 ? hx : (s == 3 ? xy : hy);
    };
    int a = lab[0], b = lab[1], c = lab[2];
    return venn_code(n[a], n[b], n[c], pr(a, b), pr(b, c), pr(c, a), hxy);
}

__device__ __forceinline__ bool within(int64_t a, int64_t b, int64_t c, int64_t w) {
    int64_t mx = a > b ? a : b, mn = a < b ? a : b;
    mx = mx > c ? mx : c;
    mn = mn < c ? mn : c;
    return mx - mn <= w;
}

// ---- hashing --------------------------------------------------------------
// Adds inc to key's value; false when every slot holds another key (the table
// is too small for the keys offered to it).
__device__ __forceinline__ bool hash_add_ok(uint32_t* keys, uint32_t* vals, uint32_t log_cap, uint32_t key,
                                            uint32_t inc) {
    uint32_t mask = (1u << log_cap) - 1u;
    uint32_t s = hash_slot(key, log_cap);
    for (uint32_t probe = 0; probe <= mask; probe++) {
        uint32_t k = __atomic_load_n(&keys[s], __ATOMIC_RELAXED);
        if (k == HGT_EMPTY) {
            uint32_t prev = atomicCAS(&keys[s], HGT_EMPTY, key);
            if (prev == HGT_EMPTY || prev == key) { atomicAdd(&vals[s], inc); return true; }
        } else if (k == key) {
            atomicAdd(&vals[s], inc);
            return true;
        }
        s = (s + 1) & mask;
    }
    return false;
}

// For tables sized for at least twice the keys offered (cannot fill up).
__device__ __forceinline__ void hash_add(uint32_t* keys, uint32_t* vals, uint32_t log_cap, uint32_t key, uint32_t inc) {
    (void)hash_add_ok(keys, vals, log_cap, key, inc);
}

// A second hash of a key, independent of hash_slot's, that splits keys into parts.
__device__ __forceinline__ uint32_t part_hash(uint32_t key) {
    uint32_t h = key * 0xcc9e2d51u;
    h ^= h >> 15;
    h *= 0x1b873593u;
    h ^= h >> 13;
    return h;
}

// returns slot index or HGT_EMPTY.  The keys are read as atomics: a table in
// global memory was filled by atomics, which bypass the CU's L1 cache.
__device__ __forceinline__ uint32_t hash_find(const uint32_t* keys, uint32_t log_cap, uint32_t key) {
    uint32_t mask = (1u << log_cap) - 1u;
    uint32_t s = hash_slot(key, log_cap);
    for (uint32_t probe = 0; probe <= mask; probe++) {
        uint32_t k = __atomic_load_n(&keys[s], __ATOMIC_RELAXED);
        if (k == key) return s;
        if (k == HGT_EMPTY) return HGT_EMPTY;
        s = (s + 1) & mask;
    }
    return HGT_EMPTY;
}


__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Work queues.  Every take is an atomic on one address that all eight L2s share, and
// such atomics pass at about 13 ns each whatever else runs (183k takes: 3.0 ms of a
// kernel of small items), so a group takes several items at once where there are many:
// at least `rounds` takes per group remain, for the balance.
__device__ __forceinline__ uint32_t take_size(uint64_t n, uint32_t groups, uint32_t rounds = 8) {
    const uint64_t c = n / ((uint64_t)rounds * groups);
    return c < 1 ? 1u : c > 16 ? 16u : (uint32_t)c;
}

// Segments laid end to end, walked by one wave: lane l holds a segment of d entries
// (0: none) and the lanes take the entries 64 at a time, so short segments fill the
// wave and no lane waits for a longer one.  The segment of an entry comes from a
// bitmap of the segments' starts (a broadcast read and a bit count instead of a binary
// search).  v = load(l, r) fetches entry r of lane l's segment, U steps' worth before
// any is used; use(ok, l, r, p, v) is called by all lanes together (ok: the lane has an
// entry; p: its number over all segments).  Returns the number of entries.
struct Flat {
    uint32_t bits[128];  // starts within the window of 4096 entries, each one place early
    uint32_t pre[64], own[64];
};
// Lays the segments out; their entries are then walked any number of times.
struct FlatSeg {
    uint32_t d, ex, tot;
};
__device__ __forceinline__ FlatSeg flat_lay(Flat& F, uint32_t d) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t inc = d;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += t;
    }
    const FlatSeg g{d, inc - d, (uint32_t)__builtin_amdgcn_readlane(inc, 63)};
    const uint64_t nz = __ballot(d != 0);
    if (d) {
        const uint32_t rank = __popcll(nz & ((1ull << lane) - 1));
        F.pre[rank] = g.ex;
        F.own[rank] = lane;
    }
    return g;
}
// The starts within the window of entries [w0, w0 + 4096).
__device__ __forceinline__ void flat_window(Flat& F, const FlatSeg& g, uint32_t w0) {
    const uint32_t lane = threadIdx.x & 63;
    F.bits[lane] = 0;
    F.bits[lane + 64] = 0;
    wave_sync();
    if (g.d && g.ex > w0 && g.ex - w0 <= 4096) atomicOr(&F.bits[(g.ex - 1 - w0) >> 5], 1u << ((g.ex - 1 - w0) & 31));
    wave_sync();
}
// use(ok, l, v) takes a lane's U entries together, so that what it fetches for one does
// not wait for the others.
template <int U, class Load, class Use>
__device__ __forceinline__ void flat_walk_all(const Flat& F, const FlatSeg& g, uint32_t w0, Load load, Use use) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t kb = (uint32_t)__popcll(__ballot(g.d && g.ex <= w0)) - 1;  // the segment that entry w0 lies in
    const uint32_t w1 = g.tot - w0 < 4096 ? g.tot : w0 + 4096;
    for (uint32_t p0 = w0; p0 < w1; p0 += 64 * U) {
        uint32_t l[U];
        bool ok[U];
        decltype(load(0u, 0u)) v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t p = p0 + 64 * u + lane, at = (p0 - w0) / 32 + 2 * u;
            const uint32_t lo = __builtin_amdgcn_readfirstlane(F.bits[at & 127]);
            const uint32_t hi = __builtin_amdgcn_readfirstlane(F.bits[(at + 1) & 127]);
            const uint32_t k = kb + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
            kb += __popc(lo) + __popc(hi);
            v[u] = {};
            l[u] = 0;
            ok[u] = p < w1;
            if (ok[u]) {
                l[u] = F.own[k];
                v[u] = load(l[u], p - F.pre[k]);
            }
        }
        use(ok, l, v);
    }
}
template <int U, class Load, class Use>
__device__ __forceinline__ void flat_walk(const Flat& F, const FlatSeg& g, uint32_t w0, Load load, Use use) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t kb = (uint32_t)__popcll(__ballot(g.d && g.ex <= w0)) - 1;  // the segment that entry w0 lies in
    const uint32_t w1 = g.tot - w0 < 4096 ? g.tot : w0 + 4096;
    for (uint32_t p0 = w0; p0 < w1; p0 += 64 * U) {
        uint32_t l[U], r[U];
        decltype(load(0u, 0u)) v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t p = p0 + 64 * u + lane, at = (p0 - w0) / 32 + 2 * u;
            const uint32_t lo = __builtin_amdgcn_readfirstlane(F.bits[at & 127]);
            const uint32_t hi = __builtin_amdgcn_readfirstlane(F.bits[(at + 1) & 127]);
            const uint32_t k = kb + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
            kb += __popc(lo) + __popc(hi);
            v[u] = {};
            l[u] = 0;
            r[u] = 0;
            if (p < w1) {
                l[u] = F.own[k];
                r[u] = p - F.pre[k];
                v[u] = load(l[u], r[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t p = p0 + 64 * u + lane;
            if (p0 + 64 * u < w1) use(p < w1, l[u], r[u], p, v[u]);
        }
    }
}
template <int U, class Load, class Use>
__device__ __forceinline__ uint32_t wave_flat(Flat& F, uint32_t d, Load load, Use use) {
    const FlatSeg g = flat_lay(F, d);
    for (uint32_t w0 = 0; w0 < g.tot; w0 += 4096) {
        flat_window(F, g, w0);
        flat_walk<U>(F, g, w0, load, use);
        wave_sync();
    }
    return g.tot;
}

// exclusive workgroup scan of one u32 per thread (all threads participate)
__device__ __forceinline__ uint32_t wg_scan_u32(uint32_t v, uint32_t* ws, uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(x, o, 64);
        if (lane >= o) x += t;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVE; w++) {
        uint32_t s = ws[w];
        if (w < wave) pre += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return pre + x - v;
}


// The slice of a sliced centre that owns neighbour x (a property of x alone, so
// every slice, whatever order its lists come in, agrees on it).
__device__ __forceinline__ uint32_t slice_of(uint32_t x, uint32_t nslice) {
    return (uint32_t)(((uint64_t)(x * 2654435761u) * nslice) >> 32);
}

// slot of a touched vertex pair in the incident-vertex family's hash
__device__ __forceinline__ uint64_t mix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

// owners: first pair index of every distinct first vertex, and of every IV_SPLIT-th pair,
// so that an owner of many pairs is shared among waves (each builds its map: a few
// hundred members against up to 64 scans)
constexpr uint64_t IV_SPLIT = 64;
__device__ __forceinline__ bool iv_head(const uint64_t* pairs, uint64_t i) {
    return i % IV_SPLIT == 0 || (pairs[i] >> 32) != (pairs[i - 1] >> 32);
}

struct Tables {
    uint8_t he[128];
    uint8_t tmp[128];
};

__device__ __forceinline__ void acc_add(uint64_t* acc, int cls, uint64_t v) {
    if (cls < 255) atomicAdd((unsigned long long*)&acc[cls], (unsigned long long)v);
}


}  // namespace tri
