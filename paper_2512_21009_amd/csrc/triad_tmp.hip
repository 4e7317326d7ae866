// triad_tmp.hip -- open paths of the temporal family, per middle hyperedge.
//
// The temporal triads {h, x, y} of a changed hyperedge h are its open paths h - x - y
// (x and y meet, h and y do not) and its closed or h-centred triples.  Here every
// pair (h, y) of neighbours of x, h changed, within the time window, counts as an open
// path, whether h and y meet or not; the pair kernel of the centres (triad_he2.hip, TMP)
// counts the triples inside N(h) and takes back the paths of those whose sides meet.
//
// N(x) depends on x alone, so it is gathered once per middle hyperedge instead of once
// per (h, x): the batch-neighbour list of x names the changed hyperedges around it.  A
// workgroup takes x, hashes the entries of its members' lists that lie in x's window (the
// lists carry timestamps) in LDS, compacts the distinct neighbours with their length and
// batch rank, and runs every changed h of x over them: window, rank and order by
// comparisons, the class from a table of 6 orders x 3 bits.
//
// What bounds it: the gathers of N(x) (12 B per list entry, two lines per distinct
// neighbour) and, for x with many changed neighbours, the (h, y) loop in LDS.
#include "triad_common.h"

namespace {

using namespace tri;

// slots with a batch-neighbour list: the middle hyperedges
__global__ void __launch_bounds__(256) k_tmp_slots(const uint64_t* __restrict__ bl_cnt, uint64_t n, uint32_t* list,
                                                   uint32_t* count) {
    __shared__ uint32_t ws[4], base;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint64_t b = (uint64_t)blockIdx.x * 1024; b < n; b += (uint64_t)gridDim.x * 1024) {
        uint64_t m[4];
        uint32_t mine = 0;
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint64_t i = b + 256 * u + threadIdx.x;
            m[u] = __ballot(i < n && bl_cnt[i] != 0);
            mine += __popcll(m[u]);
        }
        if (lane == 0) ws[wave] = mine;
        __syncthreads();
        if (threadIdx.x == 0) base = ws[0] + ws[1] + ws[2] + ws[3] ? atomicAdd(count, ws[0] + ws[1] + ws[2] + ws[3]) : 0;
        __syncthreads();
        uint32_t at = base;
        for (uint32_t w = 0; w < wave; w++) at += ws[w];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (m[u] >> lane & 1) list[at + __popcll(m[u] & ((1ull << lane) - 1))] = (uint32_t)(b + 256 * u + threadIdx.x);
            at += __popcll(m[u]);
        }
        __syncthreads();
    }
}

struct PathSh {
    uint32_t slot, stop, K, KL, over, gi, cur_g;
    uint32_t len, rank, nparts, part;
    uint64_t off, bo, bn, raw;
    int64_t t;
    uint64_t seq;
};

// N(x) as arrays of KL entries, and the hash of HS slots it is made with.
struct PathTab {
    uint32_t *keys, *vals;
    int64_t* ht;
    uint32_t *y, *meta, *rank;  // meta: c | len << 14
    int64_t* t;
};

constexpr int PCOPIES = 8;
struct PathAcc {
    uint64_t cell[48 * PCOPIES];  // [order][h only, x only, y only]
    uint8_t cls[48];
};

// Class table of an open path h - x - y: order = 3 [x before h] + (y before both: 0,
// between: 1, after both: 2).
__device__ __forceinline__ int path_code(uint32_t order, uint32_t bits) {
    // arrival positions of h, x, y
    const bool xh = order >= 3;
    const uint32_t py = order % 3;
    const uint32_t p1 = py == 0 ? 1 : 0, p2 = py == 2 ? 1 : 2;  // the earlier and the later of h, x
    const uint32_t ph = xh ? p2 : p1, px = xh ? p1 : p2;
    int code = 0;
    // region bits: 1 << p alone; pairs {0,1} 8, {1,2} 16, {0,2} 32
    if (bits & 4) code |= 1 << ph;
    if (bits & 2) code |= 1 << px;
    if (bits & 1) code |= 1 << py;
    auto pair = [](uint32_t a, uint32_t b) { return a + b == 1 ? 8 : a + b == 3 ? 16 : 32; };
    return code | pair(ph, px) | pair(px, py);
}

template <int WG, bool GLOBAL>
__device__ void paths_body(const PathParams& P, const PathTab& B, uint32_t HS, uint32_t KL, const uint32_t* list,
                           uint32_t n, uint32_t* queue, uint32_t* moved, uint32_t* n_moved) {
    constexpr uint32_t NW = WG / 64;
    __shared__ PathSh sh;
    __shared__ PathAcc A;
    __shared__ Flat flat[NW];
    __shared__ uint64_t woff_all[NW][64];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Flat& fl = flat[wave];
    uint64_t* woff = woff_all[wave];
    for (uint32_t i = tid; i < 48 * PCOPIES; i += WG) A.cell[i] = 0;
    if (tid < 48) A.cls[tid] = P.tmp_tab[path_code(tid >> 3, tid & 7)];
    if (tid == 0) sh.cur_g = 0xffffffffu;
    __syncthreads();
    auto flush = [&]() {
        __syncthreads();
        if (tid < 48 && sh.cur_g != 0xffffffffu) {
            uint64_t s = 0;
            for (int c = 0; c < PCOPIES; c++) s += A.cell[tid * PCOPIES + c];
            if (s && A.cls[tid] < 255)
                atomicAdd((unsigned long long*)&P.M.graphs[sh.cur_g].out_tmp[A.cls[tid]], (unsigned long long)s);
        }
        __syncthreads();
        for (uint32_t i = tid; i < 48 * PCOPIES; i += WG) A.cell[i] = 0;
        __syncthreads();
    };
    auto ld = [](const uint32_t* p) {
        if (GLOBAL) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return *p;
    };
    const uint32_t take = take_size(n, gridDim.x);
    uint32_t q = 0, q_end = 0;
    for (;;) {
        if (tid == 0) {
            if (q == q_end) {
                q = atomicAdd(queue, take);
                q_end = q + take;
            }
            sh.stop = q >= n;
            if (!sh.stop) {
                const uint32_t slot = list[q++];
                const uint32_t gi = multi_graph_of_id(P.M, slot);
                const HeGraph& G = P.M.graphs[gi];
                const uint32_t x = (uint32_t)(slot - G.id_base);
                sh.slot = slot;
                sh.gi = gi;
                sh.len = *((volatile const int32_t*)G.status) ? 0 : G.g.h_len[x];
                sh.off = G.g.h_off[x];
                sh.t = G.g.h_ts[x];
                sh.seq = G.g.h_seq[x];
                const uint64_t mk = G.mark[x];
                sh.rank = (uint32_t)(mk >> 32) == G.epoch ? (uint32_t)mk : 0xffffffffu;
                sh.bo = P.bl_off[slot];
                sh.bn = P.bl_cnt[slot];
                sh.raw = 0;
            }
        }
        __syncthreads();
        if (sh.stop) break;
        if (sh.gi != sh.cur_g) {
            flush();
            if (tid == 0) sh.cur_g = sh.gi;
            __syncthreads();
        }
        const HeGraph& G = P.M.graphs[sh.gi];
        const uint32_t len = sh.len, x = (uint32_t)(sh.slot - G.id_base);
        const int64_t tx = sh.t, lo = ts_sub(tx, G.window), hi = ts_add(tx, G.window);
        const uint32_t per = len / NW + 1 < 64 ? len / NW + 1 : 64;
        // entries of x's members' lists in x's window: fn(y, t)
        auto entries = [&](auto fn) {
            for (uint32_t c0 = wave * per; c0 < len; c0 += NW * per) {
                uint32_t d = 0;
                if (lane < per && c0 + lane < len) {
                    const uint32_t v = G.g.h2v[sh.off + c0 + lane];
                    d = G.g.v_len[v];
                    woff[lane] = G.g.v_off[v];
                }
                struct E {
                    int64_t t;
                    uint32_t y;
                };
                wave_flat<4>(fl, d,
                             [&](uint32_t l, uint32_t r) {
                                 const uint64_t at = woff[l] + r;
                                 return E{G.g.v2h_ts[at], G.g.v2h[at]};
                             },
                             [&](bool ok, uint32_t, uint32_t, uint32_t, E e) {
                                 if (ok && e.t >= lo && e.t <= hi && e.y != x) fn(e.y, e.t);
                             });
            }
        };
        // the largest neighbourhoods are taken in parts of the neighbours, by a second hash
        // of the ID, each part at most a quarter of the table
        uint32_t nparts = 1;
        if (GLOBAL) {
            uint64_t c = 0;
            entries([&](uint32_t, int64_t) { c++; });
            if (c) atomicAdd((unsigned long long*)&sh.raw, (unsigned long long)c);
            __syncthreads();
            const uint64_t raw = sh.raw;
            while ((uint64_t)nparts * (HS / 4) < raw) nparts <<= 1;
        }
        if (P.stats && tid == 0)
            atomicAdd((unsigned long long*)&P.stats[ST_BYTES_SMALL], (unsigned long long)(4ull * len + 16ull * sh.bn));
        for (uint32_t part = 0; part < nparts && len; part++) {
            __syncthreads();
            if (tid == 0) sh.K = sh.KL = sh.over = 0;
            for (uint32_t s = tid; s < HS; s += WG) {
                B.keys[s] = HGT_EMPTY;
                B.vals[s] = 0;
            }
            __syncthreads();
            entries([&](uint32_t y, int64_t t) {
                if (nparts > 1 && (part_hash(y) & (nparts - 1)) != part) return;
                if (*(volatile uint32_t*)&sh.K > KL) return;  // it will be moved on
                uint32_t s = (uint32_t)(((uint64_t)(y * 2654435761u) * HS) >> 32);
                for (uint32_t probe = 0; probe < HS; probe++) {
                    uint32_t k = __atomic_load_n(&B.keys[s], __ATOMIC_RELAXED);
                    if (k == HGT_EMPTY) {
                        k = atomicCAS(&B.keys[s], HGT_EMPTY, y);
                        if (k == HGT_EMPTY) {
                            B.ht[s] = t;
                            atomicAdd(&sh.K, 1u);
                            k = y;
                        }
                    }
                    if (k == y) {
                        atomicAdd(&B.vals[s], 1u);
                        return;
                    }
                    s = s + 1 == HS ? 0 : s + 1;
                }
                sh.over = 1;
            });
            __syncthreads();
            if (sh.K > KL || sh.over) {
                if (GLOBAL) {  // a part of a quarter of the table on average fills it: cannot happen
                    if (tid == 0) set_status(const_cast<int32_t*>(G.status), HGT_EDEVICE);
                } else if (tid == 0) {
                    moved[atomicAdd(n_moved, 1u)] = sh.slot;
                }
                break;
            }
            // the distinct neighbours with length and batch rank
            for (uint32_t s0 = 0; s0 < HS; s0 += WG) {
                const uint32_t s = s0 + tid;
                const uint32_t y = s < HS ? ld(&B.keys[s]) : HGT_EMPTY;
                const uint64_t m = __ballot(y != HGT_EMPTY);
                if (!m) continue;
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&sh.KL, (uint32_t)__popcll(m));
                at = __shfl(at, 0, 64) + __popcll(m & ((1ull << lane) - 1));
                if (y == HGT_EMPTY) continue;
                const uint64_t mk = G.mark[y];
                B.y[at] = y;
                B.meta[at] = ld(&B.vals[s]) | G.g.h_len[y] << 14;
                B.rank[at] = (uint32_t)(mk >> 32) == G.epoch ? (uint32_t)mk : 0xffffffffu;
                B.t[at] = B.ht[s];
            }
            __syncthreads();
            const uint32_t K = sh.KL;
            // every changed hyperedge h around x against every neighbour y
            const uint64_t bn = sh.bn;
            const uint32_t pb = bn / NW + 1 < 64 ? (uint32_t)(bn / NW) + 1 : 64;
            for (uint64_t b0 = (uint64_t)wave * pb; b0 < bn; b0 += (uint64_t)NW * pb) {
                const uint32_t nb = bn - b0 < pb ? (uint32_t)(bn - b0) : pb;
                uint32_t h_l = 0, r_l = 0, m_l = 0;
                int64_t t_l = 0;
                if (lane < nb) {
                    const uint64_t pay = P.bl_pay[sh.bo + b0 + lane];
                    h_l = P.bl_d[sh.bo + b0 + lane];
                    r_l = (uint32_t)(pay >> 32);
                    m_l = (uint32_t)(pay >> 1) & 0x3fffu;
                    m_l |= G.g.h_len[h_l] << 14;
                    t_l = G.g.h_ts[h_l];
                }
                for (uint32_t r = 0; r < nb; r++) {
                    const uint32_t h = __builtin_amdgcn_readlane(h_l, r), rh = __builtin_amdgcn_readlane(r_l, r);
                    const uint32_t mh = __builtin_amdgcn_readlane(m_l, r);
                    const int64_t th = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)t_l, r) |
                                                 (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)t_l >> 32), r)
                                                     << 32);
                    if (sh.rank < rh) continue;  // x is a batch member before h
                    const uint32_t c = mh & 0x3fffu, hlen = mh >> 14;
                    // within the window of both (the list holds those in x's)
                    const int64_t w_lo = ts_sub(th > tx ? th : tx, G.window), w_hi = ts_add(th < tx ? th : tx, G.window);
                    uint64_t sqh = 0;
                    bool xh = tx < th;  // x before h
                    if (tx == th) {
                        sqh = G.g.h_seq[h];
                        xh = sh.seq < sqh;
                    }
                    const int64_t t0 = xh ? tx : th, t1 = xh ? th : tx;  // the earlier and the later
                    const uint32_t o_base = xh ? 24 : 0, hb = hlen > c ? 4u : 0u;
                    for (uint32_t i = lane; i < K; i += 64) {
                        const int64_t ty = B.t[i];
                        const uint32_t y = B.y[i], my = B.meta[i];
                        if (y == h || ty < w_lo || ty > w_hi || B.rank[i] < rh) continue;
                        bool after0 = ty > t0, after1 = ty > t1;
                        if (ty == t0 || ty == t1) {  // ties: by arrival sequence
                            const uint64_t sy = G.g.h_seq[y], s_h = G.g.h_seq[h];
                            const uint64_t s0 = xh ? sh.seq : s_h, s1 = xh ? s_h : sh.seq;
                            if (ty == t0) after0 = sy > s0;
                            if (ty == t1) after1 = sy > s1;
                        }
                        const uint32_t cxy = my & 0x3fffu, ny = my >> 14;
                        const uint32_t cell = o_base + (after0 ? (after1 ? 16u : 8u) : 0u) + hb +
                                              (len > c + cxy ? 2u : 0u) + (ny > cxy ? 1u : 0u);
                        atomicAdd((unsigned long long*)&A.cell[cell * PCOPIES + (lane & (PCOPIES - 1))], 1ull);
                    }
                }
            }
        }
        __syncthreads();
    }
    flush();
}

constexpr uint32_t HS_S = 768, KL_S = 512;     // 256 threads, five workgroups per CU
constexpr uint32_t HS_M = 3072, KL_M = 2048;   // 512 threads, one workgroup per CU

template <int WG, uint32_t HS, uint32_t KL>
__device__ __forceinline__ void paths_lds(const PathParams& P, const uint32_t* list, uint32_t n, uint32_t* queue,
                                          uint32_t* moved, uint32_t* n_moved) {
    __shared__ int64_t ht[HS], t[KL];
    __shared__ uint32_t keys[HS], vals[HS], y[KL], meta[KL], rank[KL];
    paths_body<WG, false>(P, PathTab{keys, vals, ht, y, meta, rank, t}, HS, KL, list, n, queue, moved, n_moved);
}

__global__ void __launch_bounds__(256) k_tmp_paths(PathParams P) {
    paths_lds<256, HS_S, KL_S>(P, P.list[0], P.count[0], &P.queue[0], P.list[1], &P.count[1]);
}

__global__ void __launch_bounds__(512) k_tmp_paths_mid(PathParams P) {
    paths_lds<512, HS_M, KL_M>(P, P.list[1], P.count[1], &P.queue[1], P.list[0], &P.count[2]);
}

// the rest: tables in global memory, hash of HS slots and a list of HS entries (9 words a slot)
__global__ void __launch_bounds__(512) k_tmp_paths_global(PathParams P) {
    const uint32_t HS = (uint32_t)(P.words / 10);
    uint32_t* p = P.scratch + (uint64_t)blockIdx.x * P.words;
    int64_t* ht = (int64_t*)p;
    int64_t* t = ht + HS;
    uint32_t* u = (uint32_t*)(t + HS);
    paths_body<512, true>(P, PathTab{u, u + HS, ht, u + 2 * (uint64_t)HS, u + 3 * (uint64_t)HS, u + 4 * (uint64_t)HS, t}, HS,
                          HS - 1, P.list[0], P.count[2], &P.queue[2], nullptr, nullptr);
}

}  // namespace

void tmp_paths_launch(PathParams& P, unsigned n_cu, unsigned grid_global, hipStream_t s) {
    hgt_fill_u32(P.queue, 0, 6, s);  // three queues, three counts
    const uint64_t n = P.M.total_ids;
    const unsigned blk = (unsigned)((n + 1023) / 1024);
    k_tmp_slots<<<blk < 4 * n_cu ? blk : 4 * n_cu, 256, 0, s>>>(P.bl_cnt, n, P.list[0], &P.count[0]);
    const unsigned most = (unsigned)(n < 0xffffffu ? n : 0xffffffu);
    k_tmp_paths<<<most < 5 * n_cu ? most : 5 * n_cu, 256, 0, s>>>(P);
    k_tmp_paths_mid<<<most < n_cu ? most : n_cu, 512, 0, s>>>(P);
    k_tmp_paths_global<<<grid_global, 512, 0, s>>>(P);
}
