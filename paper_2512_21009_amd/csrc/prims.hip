// prims.hip -- device-wide exclusive scan and LSD radix sort for gfx950.
//
// Both work on tiles of 2048 elements with 256-thread workgroups (four wave64s).  Counts
// may live in device memory (n_dev): the host launches with an upper bound and no
// synchronisation, at most MAX_BLOCKS workgroups, and each takes an equal run of the
// tiles that there really are, so neither the passes nor the tables between them grow
// with the bound.  A scan is two launches (one for a single tile) and a radix pass three
// (two for few workgroups): what small inputs pay for.  With a workgroup, a table row and
// a further scan per tile of the bound, and five launches a pass, a batch of 25k + 25k changes
// on 20M hyperedges (a bound of all their 64M incidences) took 8.1 ms in all against 6.3, and
// one of 50k + 50k changes on 8M edges 2.98 ms against 2.59.
#include "hgt_dev.h"

namespace {

constexpr int ITEMS = 8;
constexpr int TILE = HGT_WG * ITEMS;  // 2048
constexpr uint32_t MAX_BLOCKS = 1024;  // four per CU
constexpr uint32_t SUM_BLOCKS = 32;    // up to these a radix pass sums the counts as it scatters

__device__ __forceinline__ uint64_t read_n(const uint64_t* n_dev, uint64_t n_max) {
    if (!n_dev) return n_max;
    uint64_t n = *n_dev;
    return n < n_max ? n : n_max;
}

// Exclusive scan of one value per thread across the workgroup.
__device__ __forceinline__ uint64_t wg_exclusive(uint64_t v, uint64_t* wave_sums, uint64_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint64_t t = __shfl_up(x, o, 64);
        if (lane >= o) x += t;
    }
    if (lane == 63) wave_sums[wave] = x;
    __syncthreads();
    uint64_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < HGT_WG / 64; w++) {
        uint64_t s = wave_sums[w];
        if (w < wave) pre += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return pre + x - v;
}

// The tiles [first, last) of this workgroup.
struct Run {
    uint64_t first, last;
};
__device__ __forceinline__ Run tiles_of_block(uint64_t n) {
    const uint64_t tiles = (n + TILE - 1) / TILE, per = (tiles + gridDim.x - 1) / gridDim.x;
    const uint64_t a = blockIdx.x * per, b = a + per;
    return Run{a < tiles ? a : tiles, b < tiles ? b : tiles};
}

__global__ void __launch_bounds__(HGT_WG) k_scan_reduce(const uint64_t* __restrict__ in, uint64_t n_max,
                                                        const uint64_t* n_dev, uint64_t* __restrict__ sums) {
    __shared__ uint64_t ws[HGT_WG / 64];
    const uint64_t n = read_n(n_dev, n_max);
    const Run r = tiles_of_block(n);
    uint64_t s = 0;
    for (uint64_t t = r.first; t < r.last; t++) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint64_t e = t * TILE + (uint64_t)i * HGT_WG + threadIdx.x;
            if (e < n) s += in[e];
        }
    }
    uint64_t tot;
    wg_exclusive(s, ws, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// sums: of every workgroup, NULL when there is one
__global__ void __launch_bounds__(HGT_WG) k_scan_down(const uint64_t* in, uint64_t* out, uint64_t n_max,
                                                      const uint64_t* n_dev, const uint64_t* __restrict__ sums,
                                                      uint64_t* total) {
    __shared__ uint64_t buf[TILE];
    __shared__ uint64_t ws[HGT_WG / 64];
    const uint64_t n = read_n(n_dev, n_max);
    const Run r = tiles_of_block(n);
    uint64_t carry = 0, all = 0;
    if (sums) {
        uint64_t before = 0, every = 0;
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += HGT_WG) {
            const uint64_t v = sums[b];
            every += v;
            if (b < blockIdx.x) before += v;
        }
        wg_exclusive(before, ws, &carry);
        wg_exclusive(every, ws, &all);
    }
    for (uint64_t t = r.first; t < r.last; t++) {
        const uint64_t base = t * TILE;
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {  // striped, coalesced load
            const uint64_t e = base + (uint64_t)i * HGT_WG + threadIdx.x;
            buf[i * HGT_WG + threadIdx.x] = e < n ? in[e] : 0;
        }
        __syncthreads();
        uint64_t loc[ITEMS];
        uint64_t s = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {  // blocked per thread
            loc[i] = s;
            s += buf[threadIdx.x * ITEMS + i];
        }
        uint64_t tot;
        const uint64_t pre = carry + wg_exclusive(s, ws, &tot);
#pragma unroll
        for (int i = 0; i < ITEMS; i++) buf[threadIdx.x * ITEMS + i] = pre + loc[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint64_t e = base + (uint64_t)i * HGT_WG + threadIdx.x;
            if (e < n) out[e] = buf[i * HGT_WG + threadIdx.x];
        }
        carry += tot;
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && total) *total = sums ? all : carry;
}

// ---- radix sort --------------------------------------------------------
constexpr int RADIX = 256;

// hist[digit * workgroups + workgroup]
__global__ void __launch_bounds__(HGT_WG) k_rs_hist(const uint64_t* __restrict__ keys, uint64_t n_max,
                                                    const uint64_t* n_dev, int shift, uint64_t* __restrict__ hist) {
    __shared__ uint32_t h[RADIX];
    const uint64_t n = read_n(n_dev, n_max);
    const Run r = tiles_of_block(n);
    uint64_t sum = 0;
    for (uint64_t t = r.first; t < r.last; t++) {
        h[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint64_t e = t * TILE + (uint64_t)i * HGT_WG + threadIdx.x;
            if (e < n) atomicAdd(&h[(keys[e] >> shift) & (RADIX - 1)], 1u);
        }
        __syncthreads();
        sum += h[threadIdx.x];
    }
    hist[(uint64_t)threadIdx.x * gridDim.x + blockIdx.x] = sum;
}

// One workgroup per digit: the exclusive scan of its counts over the workgroups, in place,
// and their sum.
__global__ void __launch_bounds__(HGT_WG) k_rs_rows(uint64_t* __restrict__ hist, uint32_t n_blocks,
                                                    uint64_t* __restrict__ digit) {
    __shared__ uint64_t ws[HGT_WG / 64];
    constexpr uint32_t PER = MAX_BLOCKS / HGT_WG;
    uint64_t* row = hist + (uint64_t)blockIdx.x * n_blocks;
    uint64_t v[PER], s = 0, tot;
#pragma unroll
    for (uint32_t i = 0; i < PER; i++) {
        const uint32_t b = threadIdx.x * PER + i;
        v[i] = b < n_blocks ? row[b] : 0;
        s += v[i];
    }
    uint64_t pre = wg_exclusive(s, ws, &tot);
#pragma unroll
    for (uint32_t i = 0; i < PER; i++) {
        const uint32_t b = threadIdx.x * PER + i;
        if (b < n_blocks) row[b] = pre;
        pre += v[i];
    }
    if (threadIdx.x == 0) digit[blockIdx.x] = tot;
}

// digit: the digits' sums, hist then holding scanned rows; NULL: a thread sums its digit's row
__global__ void __launch_bounds__(HGT_WG) k_rs_scatter(const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                                                       uint64_t n_max, const uint64_t* n_dev, int shift,
                                                       const uint64_t* __restrict__ hist,
                                                       const uint64_t* __restrict__ digit) {
    __shared__ uint64_t base_d[RADIX];
    __shared__ uint32_t wcnt[HGT_WG / 64][RADIX];
    __shared__ uint64_t ws[HGT_WG / 64];
    const uint64_t n = read_n(n_dev, n_max);
    const Run r = tiles_of_block(n);
    if (r.first >= r.last) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t* row = hist + (uint64_t)threadIdx.x * gridDim.x;
    uint64_t mine = 0, sum = 0;
    if (digit) {
        mine = row[blockIdx.x];
        sum = digit[threadIdx.x];
    } else {
        for (uint32_t b = 0; b < gridDim.x; b++) {
            const uint64_t v = row[b];
            if (b < blockIdx.x) mine += v;
            sum += v;
        }
    }
    uint64_t tot;
    base_d[threadIdx.x] = mine + wg_exclusive(sum, ws, &tot);
    const uint64_t lt_mask = (lane == 0) ? 0ull : ((1ull << lane) - 1ull);
    for (uint64_t t = r.first; t < r.last; t++) {
        uint64_t keys[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint64_t e = t * TILE + (uint64_t)i * HGT_WG + threadIdx.x;
            keys[i] = e < n ? in[e] : 0;
        }
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            for (int w = 0; w < HGT_WG / 64; w++) wcnt[w][threadIdx.x] = 0;
            __syncthreads();
            const bool valid = t * TILE + (uint64_t)i * HGT_WG + threadIdx.x < n;
            const uint64_t key = keys[i];
            const uint32_t d = (uint32_t)(key >> shift) & (RADIX - 1);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const uint64_t bb = __ballot((d >> b) & 1);
                peers &= ((d >> b) & 1) ? bb : ~bb;
            }
            const uint32_t lower = __popcll(peers & lt_mask);
            if (valid && lower == 0) wcnt[wave][d] = __popcll(peers);
            __syncthreads();
            if (valid) {
                uint32_t off = lower;
                for (int w = 0; w < wave; w++) off += wcnt[w][d];
                out[base_d[d] + off] = key;
            }
            __syncthreads();
            uint32_t add = 0;
            for (int w = 0; w < HGT_WG / 64; w++) add += wcnt[w][threadIdx.x];
            base_d[threadIdx.x] += add;
            __syncthreads();
        }
    }
}

__global__ void __launch_bounds__(HGT_WG) k_copy_live(const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                                                      uint64_t n_max, const uint64_t* n_dev) {
    const uint64_t n = read_n(n_dev, n_max);
    for (uint64_t i = (uint64_t)blockIdx.x * HGT_WG + threadIdx.x; i < n; i += (uint64_t)gridDim.x * HGT_WG) out[i] = in[i];
}

template <class T>
__global__ void k_fill(T* p, T v, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = v;
}

inline uint64_t n_blocks_of(uint64_t n) {
    const uint64_t t = (n + TILE - 1) / TILE;
    return t < MAX_BLOCKS ? t : MAX_BLOCKS;
}

}  // namespace

size_t hgt_scan_tmp_bytes(uint64_t n_max) { return (n_blocks_of(n_max) + 1) * sizeof(uint64_t); }

void hgt_scan_u64(const uint64_t* in, uint64_t* out, uint64_t n_max, const uint64_t* n_dev, uint64_t* total,
                  void* tmp, hipStream_t s) {
    const unsigned nb = (unsigned)n_blocks_of(n_max);
    uint64_t* sums = (uint64_t*)tmp;
    if (nb == 0) {
        if (total) k_fill<uint64_t><<<1, 64, 0, s>>>(total, 0, 1);
        return;
    }
    if (nb > 1) k_scan_reduce<<<nb, HGT_WG, 0, s>>>(in, n_max, n_dev, sums);
    k_scan_down<<<nb, HGT_WG, 0, s>>>(in, out, n_max, n_dev, nb > 1 ? sums : nullptr, total);
}

size_t hgt_radix_tmp_bytes(uint64_t n_max) { return (uint64_t)RADIX * (n_blocks_of(n_max) + 1) * sizeof(uint64_t); }

void hgt_radix_sort_u64(uint64_t* keys, uint64_t* alt, uint64_t n_max, const uint64_t* n_dev, int bits, void* tmp,
                        hipStream_t s) {
    const unsigned nb = (unsigned)n_blocks_of(n_max);
    if (nb == 0 || bits <= 0) return;
    uint64_t* hist = (uint64_t*)tmp;
    uint64_t* digit = nb > SUM_BLOCKS ? hist + (uint64_t)RADIX * nb : nullptr;
    const int passes = (bits + 7) / 8;
    uint64_t *src = keys, *dst = alt;
    for (int p = 0; p < passes; p++) {
        const int shift = 8 * p;
        k_rs_hist<<<nb, HGT_WG, 0, s>>>(src, n_max, n_dev, shift, hist);
        if (digit) k_rs_rows<<<RADIX, HGT_WG, 0, s>>>(hist, nb, digit);
        k_rs_scatter<<<nb, HGT_WG, 0, s>>>(src, dst, n_max, n_dev, shift, hist, digit);
        uint64_t* t = src; src = dst; dst = t;
    }
    if (src != keys) k_copy_live<<<nb, HGT_WG, 0, s>>>(src, keys, n_max, n_dev);
}

void hgt_fill_u64(uint64_t* p, uint64_t v, uint64_t n, hipStream_t s) {
    if (!n) return;
    uint64_t g = (n + 255) / 256;
    k_fill<uint64_t><<<(unsigned)(g > 4096 ? 4096 : g), 256, 0, s>>>(p, v, n);
}

void hgt_fill_u32(uint32_t* p, uint32_t v, uint64_t n, hipStream_t s) {
    if (!n) return;
    uint64_t g = (n + 255) / 256;
    k_fill<uint32_t><<<(unsigned)(g > 4096 ? 4096 : g), 256, 0, s>>>(p, v, n);
}
