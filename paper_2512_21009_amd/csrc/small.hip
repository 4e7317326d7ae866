// small.hip -- the store's planning, its update and the touched vertex pairs of small
// batches, one workgroup per graph and one launch for several graphs.
//
// What bounds small batches is the number of dependent launches (about 5 us each on the
// device, 3 us on the host): kernel by kernel, planning takes 40 of them per graph, the
// update 10, the pair list 80, and a round over many graphs pays for each graph.  Here a
// workgroup of 1024 threads does each of the three, its keys, sorts and scans in LDS
// (150 KB: one workgroup per CU, so up to 256 graphs run at once).  The
// steps, their results and their errors are those of store.hip and triad_iv.hip.
// Against those, with the counting kernels the same: one change on 20k hyperedges 1.08 ->
// 0.48 ms, 64 graphs of up to 4,000 hyperedges in one round 19.4 -> 2.9 ms.
#include "small.h"
#include "triad_common.h"

namespace {

using namespace tri;

constexpr uint32_t T = 1024, NWV = T / 64;

// exclusive scan of one value per thread; *total the sum (all threads)
template <class V>
__device__ __forceinline__ V scan1024(V v, V* ws, V* total) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    V x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const V t = __shfl_up(x, o, 64);
        if (lane >= (uint32_t)o) x += t;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    V pre = 0, tot = 0;
    for (uint32_t w = 0; w < NWV; w++) {
        if (w < wave) pre += ws[w];
        tot += ws[w];
    }
    __syncthreads();
    *total = tot;
    return pre + x - v;
}

// ascending bitonic sort of n keys in LDS (room for the next power of two)
template <class V>
__device__ void sort1024(V* k, uint32_t n) {
    constexpr V top = ~(V)0;
    const uint32_t N = (uint32_t)pow2ceil64(n < 2 ? 2 : n);
    for (uint32_t i = n + threadIdx.x; i < N; i += T) k[i] = top;
    __syncthreads();
    for (uint32_t size = 2; size <= N; size <<= 1) {
        for (uint32_t st = size >> 1; st > 0; st >>= 1) {
            for (uint32_t t = threadIdx.x; t < N / 2; t += T) {
                const uint32_t i = 2 * t - (t & (st - 1)), j = i + st;
                const V a = k[i], b = k[j];
                if ((a > b) == ((i & size) == 0)) {
                    k[i] = b;
                    k[j] = a;
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ void fail(int32_t* st, int code) { atomicCAS(st, 0, code); }

struct PlanSh {
    uint64_t keys[kSmallPairs];      // pair keys; before them bitmaps and rows being sorted
    uint32_t seg[kSmallPairs + 1];   // per touched vertex: first pair | inserted pairs before it << 16
    uint32_t nlen[kSmallPairs];      // ... its new list length
    uint32_t del_off[kSmallRows + 1], ins_off[kSmallRows + 1];
    uint64_t ws[NWV];
    uint32_t ws32[NWV];
    uint16_t big[kSmallRows];
    uint32_t n_big;
    int32_t status;
    uint64_t red[4];
    BatchSummary sum;
};

__device__ void plan_one(const SmallPlan& J, PlanSh& sh) {
    const StoreDev& g = J.g;
    const BatchIn& b = J.b;
    const PlanScratch& w = J.w;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n_del = (uint32_t)b.n_del, n_ins = (uint32_t)b.n_ins, n_mem = (uint32_t)b.n_ins_members;
    const uint64_t next_id = g.sc->next_id;
    if (tid == 0) {
        sh.status = 0;
        sh.sum = BatchSummary{};
        sh.n_big = 0;
        for (int i = 0; i < 4; i++) sh.red[i] = 0;
    }
    for (uint32_t i = tid; i < J.n_acc; i += T) J.acc[i] = 0;
    __syncthreads();
    auto finish = [&]() {
        __syncthreads();
        if (tid == 0) {
            sh.sum.status = sh.status;
            g.sc->status = sh.sum.status;
            *w.sum = sh.sum;
            *J.out = sh.sum;
        }
    };
    auto bad = [&]() {  // alike for every thread: read between two barriers
        __syncthreads();
        const bool b0 = sh.status != 0;
        __syncthreads();
        return b0;
    };
    // --- deletions: live, distinct; marks and sizes
    uint64_t members = 0, pairs2 = 0;
    for (uint32_t base = 0; base < n_del; base += T) {
        const uint32_t i = base + tid;
        uint32_t d = 0;
        if (i < n_del) {
            const uint32_t id = b.del[i];
            if ((uint64_t)id >= next_id || ((g.free_bm[id >> 6] >> (id & 63)) & 1ull)) {
                fail(&sh.status, HGT_ENOENT);
            } else {
                const uint64_t old = atomicExch((unsigned long long*)&g.mark_del[id],
                                                (unsigned long long)b.epoch_del << 32 | i);
                if ((uint32_t)(old >> 32) == b.epoch_del) fail(&sh.status, HGT_EDUP);
                else d = g.h_len[id];
            }
            w.del_card[i] = d;
            pairs2 += choose2(d);
        }
        uint32_t tot;
        const uint32_t ex = scan1024(d, sh.ws32, &tot);
        if (i < n_del) sh.del_off[i] = (uint32_t)members + ex;
        members += tot;
    }
    if (pairs2) atomicAdd((unsigned long long*)&sh.red[0], (unsigned long long)pairs2);
    if (tid == 0) sh.del_off[n_del] = (uint32_t)members;
    if (bad()) return finish();
    // --- inserts: CSR, cardinalities, temporal order
    uint64_t ip2 = 0, maxc = 0;
    const uint64_t o0 = n_ins ? b.ins_off[0] : 0;
    for (uint32_t j = tid; j < n_ins; j += T) {
        const uint64_t a = b.ins_off[j], e = b.ins_off[j + 1];
        uint64_t card = 0;
        if (a < o0 || e < a || e - o0 > n_mem) {
            fail(&sh.status, HGT_EINVAL);
        } else {
            card = e - a;
            if (card < 1 || card > HGT_MAX_CARD) fail(&sh.status, HGT_EINVAL);
        }
        if (j == n_ins - 1 && e - o0 != n_mem) fail(&sh.status, HGT_EINVAL);
        const uint64_t rel = a >= o0 ? a - o0 : 0;
        w.ins_rel[j] = rel;
        sh.ins_off[j] = (uint32_t)rel;
        if (j == n_ins - 1) {
            w.ins_rel[n_ins] = n_mem;
            sh.ins_off[n_ins] = n_mem;
        }
        w.ins_card[j] = card;
        ip2 += choose2(card);
        maxc = card > maxc ? card : maxc;
        if (b.ins_ts && b.check_order) {
            if (j > 0 && b.ins_ts[j] < b.ins_ts[j - 1]) fail(&sh.status, HGT_EORDER);
            if (j == 0 && b.ins_ts[0] < g.sc->last_ts) fail(&sh.status, HGT_EORDER);
        }
        if (card > 64) sh.big[atomicAdd(&sh.n_big, 1u)] = (uint16_t)j;
    }
    if (ip2) atomicAdd((unsigned long long*)&sh.red[1], (unsigned long long)ip2);
    if (maxc) atomicMax((unsigned long long*)&sh.red[2], (unsigned long long)maxc);
    if (bad()) return finish();
    // --- rows sorted, repeats and ranges checked
    for (uint32_t j = wave; j < n_ins; j += NWV) {
        const uint32_t a = sh.ins_off[j], card = sh.ins_off[j + 1] - a;
        if (card > 64) continue;
        uint32_t v = lane < card ? b.ins_mem[a + lane] : 0xffffffffu;
#pragma unroll
        for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
            for (int s = k >> 1; s > 0; s >>= 1) {
                const uint32_t o = __shfl_xor(v, s, 64);
                const bool up = (lane & k) == 0, lower = (lane & s) == 0;
                const uint32_t mn = v < o ? v : o, mx = v < o ? o : v;
                v = (up == lower) ? mn : mx;
            }
        }
        const uint32_t nxt = __shfl_down(v, 1, 64);
        if (lane < card) {
            if (v >= g.n_vertices || (lane + 1 < card && nxt == v)) fail(&sh.status, HGT_EINVAL);
            w.canon[a + lane] = v;
        }
    }
    __syncthreads();
    for (uint32_t q = 0; q < sh.n_big; q++) {
        const uint32_t j = sh.big[q], a = sh.ins_off[j], card = sh.ins_off[j + 1] - a;
        uint32_t* buf = (uint32_t*)sh.keys;  // HGT_MAX_CARD words
        for (uint32_t i = tid; i < card; i += T) buf[i] = b.ins_mem[a + i];
        __syncthreads();
        sort1024(buf, card);
        for (uint32_t i = tid; i < card; i += T) {
            const uint32_t v = buf[i];
            if (v >= g.n_vertices || (i + 1 < card && buf[i + 1] == v)) fail(&sh.status, HGT_EINVAL);
            w.canon[a + i] = v;
        }
        __syncthreads();
    }
    if (bad()) return finish();
    // --- IDs: the j-th insert takes the j-th smallest free ID, deletions included
    uint64_t found = 0;
    if (b.forced_ids) {
        for (uint32_t j = tid; j < n_ins; j += T) {
            w.assigned[j] = b.forced_ids[j];
            g.mark_ins[b.forced_ids[j]] = (uint64_t)b.epoch_ins << 32 | j;
        }
        found = n_ins;
    } else {
        const uint64_t nw = (next_id + 63) >> 6;
        for (uint64_t w0 = 0; w0 < nw && found < n_ins; w0 += 4 * T) {
            for (uint32_t k = tid; k < 4 * T; k += T) sh.keys[k] = 0;
            __syncthreads();
            for (uint32_t i = tid; i < n_del; i += T) {
                const uint32_t id = b.del[i];
                const uint64_t at = id >> 6;
                if (at >= w0 && at < w0 + 4 * T) atomicOr((unsigned long long*)&sh.keys[at - w0], 1ull << (id & 63));
            }
            __syncthreads();
            uint64_t bits[4];
            uint32_t c = 0, tot;
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                const uint64_t at = w0 + 4 * tid + k;
                bits[k] = at < nw ? g.free_bm[at] | sh.keys[4 * tid + k] : 0;
                c += (uint32_t)__popcll(bits[k]);
            }
            uint64_t r = found + scan1024(c, sh.ws32, &tot);
#pragma unroll
            for (uint32_t k = 0; k < 4; k++)
                while (bits[k] && r < n_ins) {
                    w.assigned[r++] =
                        (uint32_t)((w0 + 4 * tid + k) * 64 + (__ffsll((unsigned long long)bits[k]) - 1));
                    bits[k] &= bits[k] - 1;
                }
            found += tot;
            __syncthreads();
        }
        for (uint32_t j = tid; j < n_ins; j += T) {
            uint32_t id;
            if (j >= found) w.assigned[j] = id = (uint32_t)(next_id + (j - found));
            else id = w.assigned[j];
            g.mark_ins[id] = (uint64_t)b.epoch_ins << 32 | j;
        }
    }
    if (tid == 0) {
        sh.sum.n_free = found;
        sh.sum.next_id_new = next_id + (n_ins > found ? n_ins - found : 0);
    }
    __syncthreads();
    // --- words of fresh h2v blocks
    uint64_t h_total = 0;
    for (uint32_t base = 0; base < n_ins; base += T) {
        const uint32_t j = base + tid;
        uint64_t need = 0;
        if (j < n_ins) {
            const uint32_t id = w.assigned[j];
            const uint64_t cap = (uint64_t)id < next_id ? g.h_cap[id] : 0, card = sh.ins_off[j + 1] - sh.ins_off[j];
            need = card > cap ? pow2ceil64(card < 4 ? 4 : card) : 0;
            w.h_need[j] = need;
        }
        uint64_t tot;
        const uint64_t ex = scan1024(need, sh.ws, &tot);
        if (j < n_ins) w.h_rel[j] = h_total + ex;
        h_total += tot;
    }
    if (tid == 0) {
        sh.sum.h2v_need = h_total;
        sh.sum.del_members = members;
        sh.sum.del_pairs2 = sh.red[0];
        sh.sum.ins_pairs2 = sh.red[1];
        sh.sum.max_ins_card = sh.red[2];
    }
    const uint64_t n_pairs64 = members + n_mem;
    if (n_pairs64 > kSmallPairs) {
        if (tid == 0) sh.sum.pad0 = 1;
        return finish();
    }
    const uint32_t np = (uint32_t)n_pairs64;
    __syncthreads();
    // --- (vertex, hyperedge, inserted) pairs, sorted; the deleted rows' list lengths in nlen
    for (uint32_t i = tid; i < n_del; i += T) sh.nlen[i] = 0;
    __syncthreads();
    for (uint32_t p = tid; p < (uint32_t)members; p += T) {
        const uint32_t i = seg_of<uint32_t>(sh.del_off, n_del, p), id = b.del[i];
        const uint32_t v = g.h2v[g.h_off[id] + (p - sh.del_off[i])];
        sh.keys[p] = ((uint64_t)v << (g.hb + 1)) | ((uint64_t)id << 1);
        atomicAdd(&sh.nlen[i], g.v_len[v]);
    }
    for (uint32_t m = tid; m < n_mem; m += T) {
        const uint32_t j = seg_of<uint32_t>(sh.ins_off, n_ins, m);
        sh.keys[members + m] = ((uint64_t)w.canon[m] << (g.hb + 1)) | ((uint64_t)w.assigned[j] << 1) | 1ull;
    }
    if (tid == 0) sh.red[0] = sh.red[1] = 0;
    __syncthreads();
    {
        uint64_t s = 0, mx = 0;
        for (uint32_t i = tid; i < n_del; i += T) {
            s += sh.nlen[i];
            mx = sh.nlen[i] > mx ? sh.nlen[i] : mx;
        }
        if (s) atomicAdd((unsigned long long*)&sh.red[0], (unsigned long long)s);
        if (mx) atomicMax((unsigned long long*)&sh.red[1], (unsigned long long)mx);
    }
    sort1024(sh.keys, np);
    if (tid == 0) {
        sh.sum.sum_lh_del = sh.red[0];
        sh.sum.max_lh_del = sh.red[1];
    }
    // --- per touched vertex
    uint32_t nt = 0, n_ip = 0;
    for (uint32_t base = 0; base < np; base += T) {
        const uint32_t i = base + tid;
        uint64_t k = 0;
        bool hd = false;
        if (i < np) {
            k = sh.keys[i];
            hd = i == 0 || (sh.keys[i - 1] >> (g.hb + 1)) != (k >> (g.hb + 1));
        }
        const uint32_t in = i < np ? (uint32_t)(k & 1) : 0;
        uint32_t tot;
        const uint32_t ex = scan1024((hd ? 1u : 0u) | in << 16, sh.ws32, &tot);  // both sums stay below 2^14
        if (i < np) {
            const uint32_t t = nt + (ex & 0xffff) + (hd ? 1 : 0) - 1, ip = n_ip + (ex >> 16);
            const uint32_t h = (uint32_t)((k >> 1) & ((1ull << g.hb) - 1));
            if (hd) {
                w.tv[t] = (uint32_t)(k >> (g.hb + 1));
                sh.seg[t] = i | ip << 16;
            }
            if (in) {
                w.I_all[ip] = h;
                w.I_t[ip] = t;
            } else {
                w.D_all[i - ip] = h;
            }
        }
        nt += tot & 0xffff;
        n_ip += tot >> 16;
    }
    __syncthreads();
    uint64_t v_total = 0, stage = 0;
    for (uint32_t base = 0; base < nt; base += T) {
        const uint32_t t = base + tid;
        uint64_t need = 0, old = 0;
        if (t < nt) {
            const uint32_t s = sh.seg[t] & 0xffff, ips = sh.seg[t] >> 16;
            const uint32_t e = t + 1 < nt ? sh.seg[t + 1] & 0xffff : np, ipe = t + 1 < nt ? sh.seg[t + 1] >> 16 : n_ip;
            const uint32_t v = (uint32_t)(sh.keys[s] >> (g.hb + 1));
            uint64_t nI = ipe - ips, nD = (e - s) - nI;
            old = g.v_len[v];
            if (nD > old) {
                fail(&sh.status, HGT_EDEVICE);
                nD = old;
            }
            const uint64_t nl = old - nD + nI;
            w.vp.dstart[t] = s - ips;
            w.vp.istart[t] = ips;
            w.vp.nD[t] = (uint32_t)nD;
            w.vp.nI[t] = (uint32_t)nI;
            w.vp.old_len[t] = old;
            w.vp.new_len[t] = (uint32_t)nl;
            sh.nlen[t] = (uint32_t)nl;
            need = nl > g.v_cap[v] ? pow2ceil64(nl < 4 ? 4 : nl) : 0;
            w.vp.need[t] = need;
        }
        uint64_t tn, to;
        const uint64_t en = scan1024(need, sh.ws, &tn), eo = scan1024(old, sh.ws, &to);
        if (t < nt) {
            w.vp.rel[t] = v_total + en;
            w.vp.stage_off[t] = stage + eo;
        }
        v_total += tn;
        stage += to;
    }
    if (tid == 0) {
        sh.sum.v2h_need = v_total;
        sh.sum.n_touched = nt;
        sh.sum.stage_words = stage;
    }
    // --- the inserted rows' new list lengths (in del_off: the deletions are done with it)
    if (tid == 0) sh.red[0] = sh.red[1] = 0;
    for (uint32_t j = tid; j < n_ins; j += T) sh.del_off[j] = 0;
    __syncthreads();
    for (uint32_t m = tid; m < n_mem; m += T) {
        const uint32_t v = w.canon[m];
        uint32_t lo = 0, hi = nt;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if ((uint32_t)(sh.keys[sh.seg[mid] & 0xffff] >> (g.hb + 1)) <= v) lo = mid;
            else hi = mid;
        }
        atomicAdd(&sh.del_off[seg_of<uint32_t>(sh.ins_off, n_ins, m)], sh.nlen[lo]);
    }
    __syncthreads();
    {
        uint64_t s = 0, mx = 0;
        for (uint32_t j = tid; j < n_ins; j += T) {
            s += sh.del_off[j];
            mx = sh.del_off[j] > mx ? sh.del_off[j] : mx;
        }
        if (s) atomicAdd((unsigned long long*)&sh.red[0], (unsigned long long)s);
        if (mx) atomicMax((unsigned long long*)&sh.red[1], (unsigned long long)mx);
    }
    __syncthreads();
    if (tid == 0) {
        sh.sum.sum_lh_ins = sh.red[0];
        sh.sum.max_lh_ins = sh.red[1];
        *w.n_free = found;
        *w.h2v_total = h_total;
        *w.n_pairs = np;
        *w.n_touched = nt;
        *w.n_ins_pairs = n_ip;
        *w.v2h_total = v_total;
        *w.stage_total = stage;
    }
    finish();
}

template <class J>
struct ByValue {
    J j[kSmallByValue];
};
struct ByPointer {
    const SmallHost* h[kSmallJobs];
};
static_assert(sizeof(ByValue<SmallPlan>) <= 4096 && sizeof(ByValue<SmallCommit>) <= 4096, "kernel arguments");

template <class J>
__device__ __forceinline__ void fetch_job(J& to, const J& from) {  // both of 8-byte words
    for (uint32_t i = threadIdx.x; i < sizeof(J) / 8; i += T) ((uint64_t*)&to)[i] = ((const uint64_t*)&from)[i];
    __syncthreads();
}

__global__ void __launch_bounds__(T) k_small_plan(ByValue<SmallPlan> A) {
    __shared__ PlanSh sh;
    plan_one(A.j[blockIdx.x], sh);
}
__global__ void __launch_bounds__(T) k_small_plan_many(ByPointer A) {
    __shared__ PlanSh sh;
    __shared__ SmallPlan J;
    fetch_job(J, A.h[blockIdx.x]->plan);
    plan_one(J, sh);
}

// ---------------------------------------------------------------------------
// the store update (as store_commit)
// ---------------------------------------------------------------------------
struct CommitSh {
    Flat flat[NWV];
    uint64_t off_a[NWV][64], off_b[NWV][64];
};
__device__ void commit_one(const SmallCommit& C, CommitSh& sh) {
    const StoreDev& g = C.g;
    const BatchIn& b = C.b;
    const PlanScratch& w = C.w;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n_del = (uint32_t)b.n_del, n_ins = (uint32_t)b.n_ins, n_mem = (uint32_t)b.n_ins_members;
    const uint32_t nt = (uint32_t)C.n_touched;
    Flat& fl = sh.flat[wave];
    uint64_t *oa = sh.off_a[wave], *ob = sh.off_b[wave];
    for (uint32_t i = tid; i < n_del; i += T) {
        const uint32_t id = b.del[i];
        atomicOr((unsigned long long*)&g.free_bm[id >> 6], 1ull << (id & 63));
        g.h_len[id] = 0;
    }
    __syncthreads();
    for (uint32_t j = tid; j < n_ins; j += T) {
        const uint32_t id = w.assigned[j];
        const uint64_t need = w.h_need[j];
        if (need) {
            g.h_off[id] = C.h_bump + w.h_rel[j];
            g.h_cap[id] = (uint32_t)need;
        }
        g.h_len[id] = (uint32_t)w.ins_card[j];
        if (g.h_ts) g.h_ts[id] = b.ins_ts ? b.ins_ts[j] : 0;
        if (!b.keep_seq) g.h_seq[id] = C.next_seq + j;
        if ((uint64_t)id < g.next_id_host)
            atomicAnd((unsigned long long*)&g.free_bm[id >> 6], ~(1ull << (id & 63)));
        if (C.out_ids) C.out_ids[j] = id;
    }
    __syncthreads();
    // rows into their blocks
    for (uint32_t j0 = wave * 64; j0 < n_ins; j0 += T) {
        uint32_t d = 0;
        if (j0 + lane < n_ins) {
            d = (uint32_t)w.ins_card[j0 + lane];
            oa[lane] = w.ins_rel[j0 + lane];
            ob[lane] = g.h_off[w.assigned[j0 + lane]];
        }
        wave_flat<4>(fl, d, [&](uint32_t l, uint32_t r) { return w.canon[oa[l] + r]; },
                     [&](bool ok, uint32_t l, uint32_t r, uint32_t, uint32_t v) {
                         if (ok) g.h2v[ob[l] + r] = v;
                     });
    }
    // old lists of the touched vertices staged, then merged into their blocks
    for (uint32_t t0 = wave * 64; t0 < nt; t0 += T) {
        uint32_t d = 0;
        if (t0 + lane < nt) {
            const uint32_t t = t0 + lane, v = w.tv[t];
            d = (uint32_t)w.vp.old_len[t];
            oa[lane] = g.v_off[v];
            ob[lane] = w.vp.stage_off[t];
            w.dst[t] = w.vp.need[t] ? C.v_bump + w.vp.rel[t] : oa[lane];
        }
        struct E {
            int64_t t;
            uint32_t e;
        };
        wave_flat<4>(fl, d,
                     [&](uint32_t l, uint32_t r) {
                         return E{g.v2h_ts ? g.v2h_ts[oa[l] + r] : 0, g.v2h[oa[l] + r]};
                     },
                     [&](bool ok, uint32_t l, uint32_t r, uint32_t, E e) {
                         if (!ok) return;
                         w.staging[ob[l] + r] = e.e;
                         if (g.v2h_ts) w.staging_ts[ob[l] + r] = e.t;
                     });
    }
    __syncthreads();
    for (uint32_t t0 = wave * 64; t0 < nt; t0 += T) {
        uint32_t d = 0;
        if (t0 + lane < nt) {
            d = (uint32_t)w.vp.old_len[t0 + lane];
            oa[lane] = w.vp.stage_off[t0 + lane];
            ob[lane] = w.dst[t0 + lane];
        }
        wave_flat<4>(fl, d, [&](uint32_t l, uint32_t r) { return w.staging[oa[l] + r]; },
                     [&](bool ok, uint32_t l, uint32_t r, uint32_t, uint32_t e) {
                         if (!ok) return;
                         const uint32_t t = t0 + l, nD = w.vp.nD[t];
                         const uint32_t* D = w.D_all + w.vp.dstart[t];
                         const uint32_t dl = lower_bound_u32(D, nD, e);
                         if (dl < nD && D[dl] == e) return;  // deleted
                         const uint64_t pos = ob[l] + (r - dl + lower_bound_u32(w.I_all + w.vp.istart[t], w.vp.nI[t], e));
                         g.v2h[pos] = e;
                         if (g.v2h_ts) g.v2h_ts[pos] = w.staging_ts[oa[l] + r];
                     });
    }
    const uint32_t n_ip = n_mem ? (uint32_t)*w.n_ins_pairs : 0;
    for (uint32_t k = tid; k < n_ip; k += T) {
        const uint32_t t = w.I_t[k], e = w.I_all[k];
        const uint64_t pos = w.dst[t] + (k - w.vp.istart[t]) +
                             lower_bound_u32(w.staging + w.vp.stage_off[t], (uint32_t)w.vp.old_len[t], e) -
                             lower_bound_u32(w.D_all + w.vp.dstart[t], w.vp.nD[t], e);
        g.v2h[pos] = e;
        if (g.v2h_ts) g.v2h_ts[pos] = g.h_ts[e];
    }
    for (uint32_t t = tid; t < nt; t += T) {
        const uint32_t v = w.tv[t];
        g.v_off[v] = w.dst[t];
        if (w.vp.need[t]) g.v_cap[v] = (uint32_t)w.vp.need[t];
        g.v_len[v] = w.vp.new_len[t];
    }
    if (tid == 0) {
        DevScalars* sc = g.sc;
        const BatchSummary* sum = w.sum;
        sc->next_id = sum->next_id_new;
        sc->h_bump += sum->h2v_need;
        sc->v_bump += sum->v2h_need;
        if (!b.keep_seq) sc->next_seq += n_ins;
        if (b.check_order && b.ins_ts && n_ins) {
            const int64_t t = b.ins_ts[n_ins - 1];
            if (t > sc->last_ts) sc->last_ts = t;
        }
        sc->n_live = sc->n_live + n_ins - n_del;
        sc->n_inc = sc->n_inc + n_mem - sum->del_members;
    }
}

__global__ void __launch_bounds__(T) k_small_commit(ByValue<SmallCommit> A) {
    __shared__ CommitSh sh;
    commit_one(A.j[blockIdx.x], sh);
}
__global__ void __launch_bounds__(T) k_small_commit_many(ByPointer A) {
    __shared__ CommitSh sh;
    __shared__ SmallCommit C;
    fetch_job(C, A.h[blockIdx.x]->commit);
    commit_one(C, sh);
}

// ---------------------------------------------------------------------------
// touched vertex pairs (as iv_prepare and iv_touched_build)
// ---------------------------------------------------------------------------
struct IvJobs {
    SmallIv j[kSmallIvJobs];
};
static_assert(sizeof(IvJobs) <= 4096, "kernel arguments");
__global__ void __launch_bounds__(T) k_small_iv(IvJobs J) {
    __shared__ uint64_t keys[kSmallPairs], uniq[kSmallPairs];
    __shared__ uint32_t off[kSmallRows];
    __shared__ uint32_t ws[NWV];
    __shared__ unsigned long long c3[2];
    const SmallIv& P = J.j[blockIdx.x];
    if (P.sc->status) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 2) c3[tid] = 0;
    // hash of the touched pairs, cleared
    for (uint64_t i = tid; i < P.tab_slots; i += T) P.tab[i] = ~0ull;
    __syncthreads();
    uint32_t nk = 0;
    for (int side = 0; side < 2; side++) {
        const uint32_t n = (uint32_t)(side ? P.n_ins : P.n_del);
        auto row = [&](uint32_t i, const uint32_t*& m) -> uint32_t {
            if (side) {
                m = P.canon + P.ins_rel[i];
                return (uint32_t)(P.ins_rel[i + 1] - P.ins_rel[i]);
            }
            m = P.h2v + P.h_off[P.del[i]];
            return P.h_len[P.del[i]];
        };
        unsigned long long s3 = 0;
        for (uint32_t base = 0; base < n; base += T) {
            const uint32_t i = base + tid;
            uint32_t d = 0;
            const uint32_t* m;
            if (i < n) d = row(i, m);
            s3 += choose3(d);
            uint32_t tot;
            const uint32_t ex = scan1024((uint32_t)choose2(d), ws, &tot);
            if (i < n) off[i] = nk + ex;
            nk += tot;
        }
        if (s3) atomicAdd(&c3[side], s3);
        __syncthreads();
        for (uint32_t i = wave; i < n; i += NWV) {
            const uint32_t* m;
            const uint32_t d = row(i, m), o = off[i];
            for (uint32_t a = lane; a < d; a += 64) {
                uint32_t at = o + a * (2 * d - a - 1) / 2;
                const uint64_t ua = (uint64_t)m[a] << 32;
                for (uint32_t b = a + 1; b < d; b++) keys[at++] = ua | m[b];
            }
        }
        __syncthreads();
    }
    if (tid < 2) P.t1[tid] = c3[tid];
    sort1024(keys, nk);
    uint32_t nu = 0;
    for (uint32_t base = 0; base < nk; base += T) {
        const uint32_t i = base + tid;
        const bool hd = i < nk && (i == 0 || keys[i] != keys[i - 1]);
        uint32_t tot;
        const uint32_t ex = scan1024(hd ? 1u : 0u, ws, &tot);
        if (hd) uniq[nu + ex] = keys[i];
        nu += tot;
    }
    __syncthreads();
    // hash, and the pairs by owner: the endpoint of higher degree
    for (uint32_t i = tid; i < nu; i += T) {
        const uint64_t k = uniq[i];
        uint64_t s = mix64(k) & (P.tab_slots - 1);
        for (uint64_t probe = 0; probe < P.tab_slots; probe++) {
            const unsigned long long prev = atomicCAS((unsigned long long*)&P.tab[s], ~0ull, (unsigned long long)k);
            if (prev == ~0ull || prev == k) break;
            s = (s + 1) & (P.tab_slots - 1);
        }
        const uint32_t lo = (uint32_t)(k >> 32), hi = (uint32_t)k;
        keys[i] = P.v_len[hi] > P.v_len[lo] ? ((uint64_t)hi << 32 | lo) : k;
    }
    __syncthreads();
    sort1024(keys, nu);
    uint32_t no = 0;
    for (uint32_t base = 0; base < nu; base += T) {
        const uint32_t i = base + tid;
        bool hd = false;
        if (i < nu) {
            P.own[i] = keys[i];
            hd = iv_head(keys, i);
        }
        uint32_t tot;
        const uint32_t ex = scan1024(hd ? 1u : 0u, ws, &tot);
        if (hd) P.owner_start[no + ex] = i;
        no += tot;
    }
    if (tid == 0) {
        P.owner_start[no] = nu;
        *P.n_owners = no;
        *P.n_uniq = nu;
    }
}

}  // namespace

void small_plan(SmallHost* const* jobs, uint32_t n, hipStream_t s) {
    if (n <= kSmallByValue) {
        ByValue<SmallPlan> A;
        for (uint32_t i = 0; i < n; i++) A.j[i] = jobs[i]->plan;
        k_small_plan<<<n, T, 0, s>>>(A);
        return;
    }
    for (uint32_t from = 0; from < n; from += kSmallJobs) {
        const uint32_t m = n - from < kSmallJobs ? n - from : kSmallJobs;
        ByPointer A;
        for (uint32_t i = 0; i < m; i++) A.h[i] = jobs[from + i];
        k_small_plan_many<<<m, T, 0, s>>>(A);
    }
}

void small_commit(SmallHost* const* jobs, uint32_t n, hipStream_t s) {
    if (n <= kSmallByValue) {
        ByValue<SmallCommit> A;
        for (uint32_t i = 0; i < n; i++) A.j[i] = jobs[i]->commit;
        k_small_commit<<<n, T, 0, s>>>(A);
        return;
    }
    for (uint32_t from = 0; from < n; from += kSmallJobs) {
        const uint32_t m = n - from < kSmallJobs ? n - from : kSmallJobs;
        ByPointer A;
        for (uint32_t i = 0; i < m; i++) A.h[i] = jobs[from + i];
        k_small_commit_many<<<m, T, 0, s>>>(A);
    }
}

void small_iv(const SmallIv* jobs, uint32_t n, hipStream_t s) {
    IvJobs J;
    for (uint32_t i = 0; i < n; i++) J.j[i] = jobs[i];
    k_small_iv<<<n, T, 0, s>>>(J);
}
