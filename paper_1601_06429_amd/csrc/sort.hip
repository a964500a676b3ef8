// sort.hip -- particle ordering for the neighbour search.
//
// Each world (item) is quantised on a 2^16 grid over a cube of side S, and its
// particles are sorted along the Morton curve (key = item << 48 | morton48) by
// an LSD radix sort with 8-bit digits, or, if few, by comparing all pairs.  A
// Morton cell at level l is then a contiguous range of the sorted arrays; a
// dense table at level T (8^T cells, about one particle per cell) gives these
// ranges directly for l <= T, and a binary search inside a level-T cell gives
// them for l > T.  This replaces the search structure the paper gets from Qhull
// (section 2) with one whose memory accesses are contiguous ranges.
#include <algorithm>

#include "vt_internal.h"

#define SORT_THREADS 512
#define SORT_ITEMS 8
#define SORT_TILE (SORT_THREADS * SORT_ITEMS)

// ------------------------------------------------------------------ scan
#define SCAN_THREADS 256
#define SCAN_ITEMS 16
#define SCAN_TILE (SCAN_THREADS * SCAN_ITEMS)

int64_t vt_scan_tmp_elems(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE + 1; }

template <typename T>
__device__ T block_exclusive_scan(T v, T *lds, T *total) {
    // Hillis-Steele over the block (256 threads) in LDS
    int t = threadIdx.x;
    lds[t] = v;
    __syncthreads();
    for (int off = 1; off < SCAN_THREADS; off <<= 1) {
        T x = (t >= off) ? lds[t - off] : T(0);
        __syncthreads();
        lds[t] += x;
        __syncthreads();
    }
    T incl = lds[t];
    *total = lds[SCAN_THREADS - 1];
    __syncthreads();
    return incl - v;
}

// Up to three arrays of one length, back to back in `in`, are scanned side by side (blockIdx.y).
template <typename T>
struct ScanOut {
    T *out[3];
};

template <typename T>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_reduce(const T *in, int64_t n, int64_t *sums) {
    __shared__ int64_t lds[SCAN_THREADS];
    in += blockIdx.y * n;
    sums += blockIdx.y * (int64_t)(gridDim.x + 1);
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t acc = 0;
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = base + (int64_t)i * SCAN_THREADS + threadIdx.x;
        if (k < n) acc += (int64_t)in[k];
    }
    int64_t tot;
    block_exclusive_scan<int64_t>(acc, lds, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// one block per array: exclusive scan of the block sums (nb <= SCAN_THREADS * 64)
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_top(int64_t *sums, int64_t nb) {
    __shared__ int64_t lds[SCAN_THREADS];
    sums += blockIdx.x * (nb + 1);
    const int per = (int)((nb + SCAN_THREADS - 1) / SCAN_THREADS);
    int64_t base = (int64_t)threadIdx.x * per;
    int64_t acc = 0;
    for (int i = 0; i < per; ++i)
        if (base + i < nb) acc += sums[base + i];
    int64_t tot;
    int64_t off = block_exclusive_scan<int64_t>(acc, lds, &tot);
    for (int i = 0; i < per; ++i)
        if (base + i < nb) {
            int64_t x = sums[base + i];
            sums[base + i] = off;
            off += x;
        }
    if (threadIdx.x == 0) sums[nb] = tot;
}

template <typename T>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_down(const T *in, ScanOut<T> O, int64_t n, const int64_t *sums,
                                                            int write_total, int64_t nb) {
    __shared__ int64_t lds[SCAN_THREADS];
    in += blockIdx.y * n;
    sums += blockIdx.y * (nb + 1);
    T *out = blockIdx.y == 0 ? O.out[0] : blockIdx.y == 1 ? O.out[1] : O.out[2];
    __shared__ T tile[SCAN_TILE];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = base + (int64_t)i * SCAN_THREADS + threadIdx.x;
        tile[i * SCAN_THREADS + threadIdx.x] = (k < n) ? in[k] : T(0);
    }
    __syncthreads();
    // each thread scans SCAN_ITEMS consecutive elements of the tile
    int64_t acc = 0;
    T loc[SCAN_ITEMS];
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        loc[i] = tile[threadIdx.x * SCAN_ITEMS + i];
        acc += (int64_t)loc[i];
    }
    int64_t tot;
    int64_t off = block_exclusive_scan<int64_t>(acc, lds, &tot) + sums[blockIdx.x];
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        tile[threadIdx.x * SCAN_ITEMS + i] = (T)off;
        off += (int64_t)loc[i];
    }
    __syncthreads();
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = base + (int64_t)i * SCAN_THREADS + threadIdx.x;
        if (k < n) out[k] = tile[i * SCAN_THREADS + threadIdx.x];
    }
    if (write_total && blockIdx.x == 0 && threadIdx.x == 0) out[n] = (T)sums[nb];
}

// a scan of at most one tile: the block's own prefix, and the total, in one launch
template <typename T>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_single(const T *in, ScanOut<T> O, int64_t n) {
    __shared__ int64_t lds[SCAN_THREADS];
    in += blockIdx.x * n;
    T *out = blockIdx.x == 0 ? O.out[0] : blockIdx.x == 1 ? O.out[1] : O.out[2];
    const int t = threadIdx.x;
    int64_t acc = 0;
    T loc[SCAN_ITEMS];
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = (int64_t)t * SCAN_ITEMS + i;
        loc[i] = k < n ? in[k] : T(0);
        acc += (int64_t)loc[i];
    }
    int64_t tot;
    int64_t off = block_exclusive_scan<int64_t>(acc, lds, &tot);
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = (int64_t)t * SCAN_ITEMS + i;
        if (k < n) out[k] = (T)off;
        off += (int64_t)loc[i];
    }
    if (t == 0) out[n] = (T)tot;
}

template <typename T>
static hipError_t scan_impl(const T *in, ScanOut<T> out, int count, int64_t n, int64_t *tmp, hipStream_t s) {
    int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb == 0) nb = 1;
    if (nb > SCAN_THREADS * 64) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nb, (unsigned)count);
    if (nb == 1) {
        k_scan_single<T><<<count, SCAN_THREADS, 0, s>>>(in, out, n);
        return hipGetLastError();
    }
    k_scan_reduce<T><<<grid, SCAN_THREADS, 0, s>>>(in, n, tmp);
    k_scan_top<<<count, SCAN_THREADS, 0, s>>>(tmp, nb);
    k_scan_down<T><<<grid, SCAN_THREADS, 0, s>>>(in, out, n, tmp, 1, nb);
    return hipGetLastError();
}

// exclusive scan: out[0..n] with out[n] = total; in and out must not overlap
hipError_t vt_launch_scan_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *tmp, hipStream_t s) {
    return scan_impl<int64_t>(in, ScanOut<int64_t>{{out, out, out}}, 1, n, tmp, s);
}
hipError_t vt_launch_scan_i32(const int32_t *in, int32_t *out, int64_t n, int64_t *tmp, hipStream_t s) {
    return scan_impl<int32_t>(in, ScanOut<int32_t>{{out, out, out}}, 1, n, tmp, s);
}
// three arrays of n, back to back in `in`; tmp holds 3 vt_scan_tmp_elems(n)
hipError_t vt_launch_scan3_i64(const int64_t *in, int64_t *o0, int64_t *o1, int64_t *o2, int64_t n, int64_t *tmp,
                               hipStream_t s) {
    return scan_impl<int64_t>(in, ScanOut<int64_t>{{o0, o1, o2}}, 3, n, tmp, s);
}

__global__ void k_zero_u32(uint32_t *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

hipError_t vt_launch_zero_u32(uint32_t *p, int64_t n, hipStream_t s) {
    k_zero_u32<<<(n + 255) / 256, 256, 0, s>>>(p, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------ keys
__device__ __forceinline__ int find_item(const DevItem *items, int n_items, int64_t p) {
    int lo = 0, hi = n_items - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (items[mid].start <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <typename PT>
__device__ __forceinline__ uint64_t particle_key(const PT *pos, int64_t p, const DevItem &it, int b) {
    uint64_t q[3];
    for (int a = 0; a < 3; ++a) {
        double x = (double)pos[3 * p + a];
        if (it.periodic) x -= it.L[a] * floor((x - it.lo[a]) / it.L[a]);
        q[a] = (uint64_t)vt_qclamp(vt_qraw(x, it.lo[a], it.inv_res));
    }
    return ((uint64_t)b << VT_LOCAL_KEY_BITS) | vt_morton(q[0], q[1], q[2]);
}

// (also clears the build's counters, the first kernel of a build: a launch less); vals: the particle
// itself, or for k_sort_count whether it is owned
template <typename PT>
__global__ void k_keys(const PT *pos, int64_t n, const DevItem *items, int n_items, uint64_t *keys, uint32_t *vals,
                       bool owned, uint32_t *counters) {
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < CTR_COUNT) counters[p] = 0u;
    if (p >= n) return;
    const int b = find_item(items, n_items, p);
    const DevItem &it = items[b];
    keys[p] = particle_key(pos, p, it, b);
    vals[p] = owned ? (uint32_t)(p - it.start < it.n_owned) : (uint32_t)p;
}

// ------------------------------------------------------------------ radix sort
// A tile's counts go to hist[digit * sd + block * sb]: by digit where the counts are scanned as one
// array, by block where the scatter sums them itself.
__global__ void __launch_bounds__(SORT_THREADS) k_radix_hist(const uint64_t *keys, int64_t n, int shift,
                                                             int32_t *hist, int64_t sd, int64_t sb) {
    __shared__ int32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = (int64_t)blockIdx.x * SORT_TILE;
    for (int i = 0; i < SORT_ITEMS; ++i) {
        int64_t k = base + (int64_t)i * SORT_THREADS + threadIdx.x;
        if (k < n) atomicAdd(&h[(keys[k] >> shift) & 255u], 1);
    }
    __syncthreads();
    if (threadIdx.x < 256) hist[threadIdx.x * sd + blockIdx.x * sb] = h[threadIdx.x];
}

// exclusive scan of one value per thread of the first 256 (the others' v is ignored); lds: 4 ints.
// Two barriers; every thread of the block calls it.
__device__ __forceinline__ int32_t digit_scan(int32_t v, int32_t *lds) {
    const int t = threadIdx.x, lane = t & 63;
    int32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (t < 256 && lane == 63) lds[t >> 6] = incl;
    __syncthreads();
    int32_t pre = incl - v;
    for (int ww = 0; ww < 3; ++ww)
        if ((t >> 6) > ww) pre += lds[ww];
    __syncthreads();
    return pre;
}

__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Stable ranks of a tile's keys by one digit.  A wavefront holds 64 x IT consecutive keys (round i,
// lane l: its key 64 i + l) and counts its digits by itself, in its own row of wcnt: the lanes with
// the same digit are found with eight ballots and the first of them moves the counter, so the rounds
// need no barrier (a counter shared by the block's wavefronts took four a round: the scatter 21 us a
// pass at 64 tiles, now 9).  One prefix over the wavefronts and one over the digits then give each key its
// slot in the tile ordered by digit.  dstart: the digits' starts in the tile; returns, in thread t <
// 256, the tile's count of digit t.
template <int NW, int IT>
__device__ __forceinline__ int32_t tile_rank(const uint64_t (&key)[IT], int cnt, int shift, uint16_t (*wcnt)[256],
                                             int32_t *lds, int32_t *dstart, int (&slot)[IT]) {
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int k = 0; k < 4; ++k) wcnt[w][64 * k + lane] = 0;
    wave_lds_order();
    for (int i = 0; i < IT; ++i) {
        const bool valid = (w * IT + i) * 64 + lane < cnt;
        const uint32_t d = (uint32_t)(key[i] >> shift) & 255u;
        uint64_t match = __ballot(valid);
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t b = __ballot((d >> bit) & 1u);
            match &= ((d >> bit) & 1u) ? b : ~b;
        }
        const int rank = __popcll(match & lt);
        const int before = wcnt[w][d];
        wave_lds_order();
        if (valid && rank == 0) wcnt[w][d] = (uint16_t)(before + __popcll(match));
        wave_lds_order();
        slot[i] = before + rank;
    }
    __syncthreads();
    int32_t tot = 0;
    if (t < 256)
        for (int ww = 0; ww < NW; ++ww) {
            const int32_t c = wcnt[ww][t];
            wcnt[ww][t] = (uint16_t)tot;
            tot += c;
        }
    const int32_t start = digit_scan(tot, lds);
    if (t < 256) dstart[t] = start;
    __syncthreads();
    for (int i = 0; i < IT; ++i) {
        const uint32_t d = (uint32_t)(key[i] >> shift) & 255u;
        slot[i] += wcnt[w][d] + dstart[d];
    }
    return tot;
}

// One pass's scatter of a tile: reordered by digit in LDS, then written out in that order, so that
// consecutive threads write consecutive slots of each digit's run (16 keys per digit on average).
// offs null: the block sums the counts of the tiles before its own itself (hist by block), both halves
// of it every other tile; else offs holds the scan of all counts (hist by digit).
__global__ void __launch_bounds__(SORT_THREADS) k_radix_scatter(const uint64_t *kin, const uint32_t *vin,
                                                                uint64_t *kout, uint32_t *vout, int64_t n,
                                                                int shift, const int32_t *hist, const int32_t *offs,
                                                                int nblocks) {
    constexpr int NW = SORT_THREADS / 64;
    __shared__ uint16_t wcnt[NW][256];
    __shared__ int32_t scan_lds[4], dstart[256], gbase[256], part[2][2][256];
    __shared__ uint64_t lkey[SORT_TILE];
    __shared__ uint32_t lval[SORT_TILE];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63, blk = (int)blockIdx.x;
    const int64_t base = (int64_t)blk * SORT_TILE, left = n - base;
    const int cnt = left < (int64_t)SORT_TILE ? (int)left : SORT_TILE;
    uint64_t key[SORT_ITEMS];
    uint32_t val[SORT_ITEMS];
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const int k = (w * SORT_ITEMS + i) * 64 + lane;
        key[i] = k < cnt ? kin[base + k] : 0ull;
        val[i] = k < cnt ? vin[base + k] : 0u;
    }
    int32_t off = 0;
    if (offs) {
        if (t < 256) off = offs[(int64_t)t * nblocks + blk];
    } else {
        const int d = t & 255, h = t >> 8;
        int32_t before = 0, all = 0;
#pragma unroll 16
        for (int b = h; b < nblocks; b += SORT_THREADS / 256) {
            const int32_t c = hist[(int64_t)b * 256 + d];
            all += c;
            before += b < blk ? c : 0;
        }
        part[0][h][d] = before;
        part[1][h][d] = all;
        __syncthreads();
        int32_t tot = 0;
        if (t < 256) {
            off = part[0][0][t] + part[0][1][t];
            tot = part[1][0][t] + part[1][1][t];
        }
        off += digit_scan(tot, scan_lds);
    }
    int slot[SORT_ITEMS];
    tile_rank<NW, SORT_ITEMS>(key, cnt, shift, wcnt, scan_lds, dstart, slot);
    if (t < 256) gbase[t] = off - dstart[t];
    for (int i = 0; i < SORT_ITEMS; ++i)
        if ((w * SORT_ITEMS + i) * 64 + lane < cnt) {
            lkey[slot[i]] = key[i];
            lval[slot[i]] = val[i];
        }
    __syncthreads();
    for (int idx = t; idx < cnt; idx += SORT_THREADS) {
        const uint64_t k = lkey[idx];
        const int32_t pos = gbase[(uint32_t)(k >> shift) & 255u] + idx;
        kout[pos] = k;
        vout[pos] = lval[idx];
    }
}

// ------------------------------------------------------------------ sorted arrays
// particle p as the j-th of the sorted arrays; returns its row (-1: not owned)
template <typename PT, typename PT4>
__device__ __forceinline__ int32_t put_sorted(const PT *pos, const int32_t *gid, int64_t p, int64_t j,
                                              const DevItem *items, int n_items, PT4 *spos, int32_t *sgid,
                                              int32_t *srow, int32_t *sorig) {
    int b = find_item(items, n_items, p);
    const DevItem &it = items[b];
    PT4 v;
    double x[3];
    for (int a = 0; a < 3; ++a) {
        x[a] = (double)pos[3 * p + a];
        if (it.periodic) {
            x[a] -= it.L[a] * floor((x[a] - it.lo[a]) / it.L[a]);
            if (x[a] >= it.lo[a] + it.L[a]) x[a] = it.lo[a];  // a value that rounds up to the top wall wraps to lo
        }
    }
    v.x = (decltype(v.x))x[0];
    v.y = (decltype(v.x))x[1];
    v.z = (decltype(v.x))x[2];
    v.w = 0;
    spos[j] = v;
    sgid[j] = gid ? gid[p] : (int32_t)p;
    int64_t k = p - it.start;
    const int32_t r = (k < it.n_owned) ? (int32_t)(it.owned_base + k) : -1;
    srow[j] = r;
    sorig[j] = (int32_t)p;
    return r;
}

// all_owned: no particle is a buffer one, so the owned cells in Morton order are the sorted particles
// and the list is written here (five launches less than flags, scan and compaction)
template <typename PT, typename PT4>
__global__ void k_sorted_gather(const PT *pos, const int32_t *gid, const uint32_t *order, int64_t n,
                                const DevItem *items, int n_items, PT4 *spos, int32_t *sgid, int32_t *srow,
                                int32_t *sorig, bool all_owned, int32_t *cells, int32_t *row2cell) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int32_t r = put_sorted(pos, gid, (int64_t)order[j], j, items, n_items, spos, sgid, srow, sorig);
    if (all_owned) {
        cells[j] = (int32_t)j;
        row2cell[r] = (int32_t)j;
    }
}

// Small inputs: every particle's place is the number of keys before its own (equal ones by input
// order), counted by comparing all pairs.  That is n^2 / 64 wavefront compares, but one launch that
// fills the chip, against two latency-bound ones for each of six radix passes.  A block places
// COUNT_KEYS keys, each wavefront counting a quarter of the input: its compares' masks are counted by
// the scalar unit, and those of owned particles give the place in the list of owned cells.  It then
// writes its particles' sorted arrays itself.  4096 particles: 11 us (a radix sort by one block, 111 us,
// or 45 with the keys kept in LDS over the passes and the gather and the list of owned cells in it).
#define COUNT_KEYS 16  // a divisor of 64: a block's keys lie in one chunk of 64
template <typename PT, typename PT4, bool ALL_OWNED>
__global__ void __launch_bounds__(256) k_sort_count(const PT *pos, const int32_t *gid, const uint64_t *keys,
                                                    const uint32_t *owned, int n, const DevItem *items,
                                                    int n_items, uint64_t *skey, PT4 *spos, int32_t *sgid,
                                                    int32_t *srow, int32_t *sorig, int32_t *cells,
                                                    int32_t *row2cell) {
    __shared__ int32_t part[2][4][COUNT_KEYS];
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int j0 = (int)blockIdx.x * COUNT_KEYS, chunk = j0 & ~63;
    uint64_t K[COUNT_KEYS];
    for (int q = 0; q < COUNT_KEYS; ++q) K[q] = keys[min(j0 + q, n - 1)];
    int32_t before[COUNT_KEYS], own[COUNT_KEYS];
    for (int q = 0; q < COUNT_KEYS; ++q) before[q] = own[q] = 0;
    auto count = [&](int base, auto below) {
        const int k = base + lane;
        const uint64_t key = k < n ? keys[k] : ~0ull;  // a key has at most 63 bits here: no padding is below one
        uint64_t mine = 0;
        if (!ALL_OWNED) {
            const uint32_t o = k < n ? owned[k] : 0u;
            mine = __ballot(o != 0);
        }
#pragma unroll
        for (int q = 0; q < COUNT_KEYS; ++q) {
            const uint64_t m = __ballot(below(key, k, q));
            before[q] += __popcll(m);
            if (!ALL_OWNED) own[q] += __popcll(m & mine);
        }
    };
    // the chunks before the block's own (an equal key goes first there), its own, those after
    int base = 64 * w;
#pragma unroll 2
    for (; base < chunk; base += 256) count(base, [&](uint64_t key, int, int q) { return key <= K[q]; });
    if (base == chunk) {
        count(base, [&](uint64_t key, int k, int q) { return key < K[q] || (key == K[q] && k < j0 + q); });
        base += 256;
    }
#pragma unroll 2
    for (; base < n; base += 256) count(base, [&](uint64_t key, int, int q) { return key < K[q]; });
    for (int q = 0; q < COUNT_KEYS; ++q)
        if (lane == q) {
            part[0][w][q] = before[q];
            part[1][w][q] = own[q];
        }
    __syncthreads();
    if (t >= COUNT_KEYS || j0 + t >= n) return;
    const int j = part[0][0][t] + part[0][1][t] + part[0][2][t] + part[0][3][t];
    const int c = ALL_OWNED ? j : part[1][0][t] + part[1][1][t] + part[1][2][t] + part[1][3][t];
    skey[j] = keys[j0 + t];
    const int32_t r = put_sorted(pos, gid, (int64_t)(j0 + t), (int64_t)j, items, n_items, spos, sgid, srow, sorig);
    if (r >= 0) {
        cells[c] = j;
        row2cell[r] = c;
    }
}

// level-T table: tab[off + c] = first sorted index whose level-T cell is >= c.  The entries from
// particle j's predecessor's cell (exclusive) to its own take j, and the last particle of an item
// also fills the rest of the item's table.  A wavefront's 64 consecutive particles own one
// contiguous stretch of the table.  When the stretch is short its lanes write it together, entry
// by entry (the value of an entry is the first of the 64 whose cell reaches it, found by a binary
// search over their cells), so the writes are coalesced however unevenly the particles fill the
// cells.  Otherwise (empty regions: voids, the part of a cuboid item's Morton cube outside the item,
// the end of an item's table) each lane writes its own run if it is short, and lists a long run
// as pieces of at most VT_TAB_PIECE entries (slots reserved once per wavefront), which k_level_fill
// writes a wavefront per piece; runs that find the list full are written by their own lane.
#define VT_TAB_STRETCH 2048
#define VT_TAB_SHORT 64
#define VT_TAB_PIECE 4096
__device__ __forceinline__ int64_t tab_pieces(int64_t len) {
    return len > VT_TAB_SHORT ? (len + VT_TAB_PIECE - 1) / VT_TAB_PIECE : 0;
}

// Each lane's runs (its own and, for an item's last particle, the tail): short ones written here,
// long ones listed in slots reserved for the whole wavefront with one atomic; a lane whose slots do
// not all fit writes its runs itself and leaves its slots below the capacity as empty pieces.
__device__ __forceinline__ void tab_runs(int32_t *tab, int64_t loA, int64_t lenA, int32_t vA, int64_t loB, int64_t lenB,
                                         int32_t vB, uint64_t *pieces, int64_t piece_cap, uint32_t *counters) {
    const int64_t pa = tab_pieces(lenA), pb = tab_pieces(lenB), mine = pa + pb;
    // inclusive prefix of the lanes' piece counts, then one reservation for the wavefront
    const int lane = (int)(threadIdx.x & 63);
    int64_t pre = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = (int64_t)__shfl_up((long long)pre, o);
        if (lane >= o) pre += y;
    }
    const int64_t total = (int64_t)__shfl((long long)pre, 63);
    pre -= mine;
    int64_t base = 0;
    if (total > 0) {
        if (lane == 0) base = (int64_t)atomicAdd(&counters[CTR_TAB_PIECES], (uint32_t)total);
        base = (int64_t)__shfl((long long)base, 0);
    }
    const int64_t k0 = base + pre;
    const bool fits = k0 + mine <= piece_cap;
    if (!fits)
        for (int64_t q = k0; q < k0 + mine && q < piece_cap; ++q) {
            pieces[2 * q] = 0;
            pieces[2 * q + 1] = 0;
        }
    auto put = [&](int64_t lo, int64_t len, int32_t v, int64_t np, int64_t k) {
        if (np == 0 || !fits) {
            for (int64_t x = 0; x < len; ++x) tab[lo + x] = v;
            return;
        }
        for (int64_t q = 0; q < np; ++q) {
            const int64_t a = q * VT_TAB_PIECE, m = len - a < VT_TAB_PIECE ? len - a : VT_TAB_PIECE;
            pieces[2 * (k + q)] = (uint64_t)(lo + a);
            pieces[2 * (k + q) + 1] = ((uint64_t)m << 32) | (uint64_t)(uint32_t)v;
        }
    };
    if (lenA > 0) put(loA, lenA, vA, pa, k0);
    if (lenB > 0) put(loB, lenB, vB, pb, k0 + pa);
}

__global__ void __launch_bounds__(256) k_level_table(const uint64_t *skey, int64_t n, const DevItem *items,
                                                     int n_items, int32_t *tab, uint64_t *pieces, int64_t piece_cap,
                                                     uint32_t *counters) {
    __shared__ int64_t cells[4][64];
    const int lane = (int)(threadIdx.x & 63), wv = (int)(threadIdx.x >> 6);
    const int64_t jw = (int64_t)blockIdx.x * blockDim.x + wv * 64;  // the wavefront's first particle
    if (jw >= n) return;
    const int64_t j = jw + lane;
    const bool valid = j < n;
    const uint64_t lmask = (1ull << VT_LOCAL_KEY_BITS) - 1;
    int b = valid ? find_item(items, n_items, j) : -1;
    int64_t c = INT64_MAX, cprev = -1;
    if (valid) {
        const DevItem &it = items[b];
        const int sh = 3 * (VT_MORTON_BITS - it.T);
        c = (int64_t)((skey[j] & lmask) >> sh);
        cprev = (j == it.start) ? -1 : (int64_t)((skey[j - 1] & lmask) >> sh);
    }
    const int b0 = __shfl(b, 0);
    const uint64_t vm = __ballot(valid);
    const int last = 63 - __builtin_clzll(vm);
    const int64_t x0 = (int64_t)__shfl((long long)cprev, 0) + 1, x1 = (int64_t)__shfl((long long)c, last);
    if (__ballot(valid && b != b0) != 0 || x1 - x0 + 1 > VT_TAB_STRETCH) {
        // the wavefront spans two items, or its stretch is long: each lane its own runs
        int64_t loA = 0, lenA = 0, loB = 0, lenB = 0;
        int32_t vB = 0;
        if (valid) {
            const DevItem &it = items[b];
            loA = it.tab_off + cprev + 1;
            lenA = c - cprev;
            if (j == it.start + it.count - 1) {
                loB = it.tab_off + c + 1;
                lenB = (1ll << (3 * it.T)) - c;
                vB = (int32_t)(it.start + it.count);
            }
        }
        tab_runs(tab, loA, lenA, (int32_t)j, loB, lenB, vB, pieces, piece_cap, counters);
        return;
    }
    const DevItem &it = items[b0];
    cells[wv][lane] = c;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int64_t x = x0 + lane; x <= x1; x += 64) {
        int lo = 0, hi = last;  // the first particle whose cell is >= x (cells ascend; the last one's is x1)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cells[wv][mid] >= x) hi = mid; else lo = mid + 1;
        }
        tab[it.tab_off + x] = (int32_t)(jw + lo);
    }
    if (jw + last == it.start + it.count - 1) {
        // the item's tail, from the lane of its last particle
        const bool mine = lane == last;
        tab_runs(tab, 0, 0, 0, mine ? it.tab_off + x1 + 1 : 0, mine ? (1ll << (3 * it.T)) - x1 : 0,
                 (int32_t)(it.start + it.count), pieces, piece_cap, counters);
    }
}

// the listed pieces, a wavefront per piece
__global__ void __launch_bounds__(256) k_level_fill(const uint64_t *pieces, int64_t piece_cap, const uint32_t *counters,
                                                    int32_t *tab) {
    const int64_t np = min((int64_t)counters[CTR_TAB_PIECES], piece_cap);
    const int lane = (int)(threadIdx.x & 63);
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t p = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); p < np; p += nw) {
        const int64_t lo = (int64_t)pieces[2 * p];
        const uint64_t w = pieces[2 * p + 1];
        const int64_t m = (int64_t)(w >> 32);
        const int32_t v = (int32_t)(uint32_t)w;
        for (int64_t x = lane; x < m; x += 64) tab[lo + x] = v;
    }
}

__global__ void k_owned_flags(const int32_t *srow, int64_t n, int32_t *flag) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) flag[j] = srow[j] >= 0 ? 1 : 0;
}

__global__ void k_owned_compact(const int32_t *srow, const int32_t *scan, int64_t n, int32_t *cells,
                                int32_t *row2cell) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    int32_t r = srow[j];
    if (r >= 0) {
        int32_t c = scan[j];
        cells[c] = (int32_t)j;
        row2cell[r] = c;
    }
}

// Up to this many tiles the blocks of the scatter sum the tiles' counts themselves, each reading all of
// them (1 KB a tile); beyond, the counts are scanned, in three launches more a pass.  Whole builds,
// summed | scanned: 300000 particles (74 tiles) 3742 | 3809 us, 600000 (147) 6946 | 7002, 1000000 (245)
// 11468 | 11520.
#define SORT_DIRECT_TILES 256
// Up to this many particles a build sorts by comparing all pairs.  Whole builds of uniform particles,
// compared | by radix passes: 4096 195 | 248 us, 16384 368 | 415, 24000 477 | 497, 32768 615 | 592;
// with a third of them buffer particles 16384 320 | 361, 24000 426 | 411.
#define SORT_COUNT_MAX 20480

template <typename PT, typename PT4>
static hipError_t launch_sort(vt_ctx *c, const PT *pos, const int32_t *gid) {
    hipStream_t s = c->stream;
    const int64_t n = c->n_total;
    const int nb = (int)((n + SORT_TILE - 1) / SORT_TILE);
    const int tpb = 256;
    const int64_t grid = (n + tpb - 1) / tpb;
    const bool all_owned = c->n_owned == n;
    if (nb > SCAN_THREADS * 64) return hipErrorInvalidValue;  // the scans' limit
    const bool count = n <= SORT_COUNT_MAX;
    k_keys<PT><<<(std::max<int64_t>(n, CTR_COUNT) + tpb - 1) / tpb, tpb, 0, s>>>(
        pos, n, c->items, c->n_items, c->keys[0], c->vals[0], count, c->counters);
    int cur = 0;
    if (count) {
        cur = 1;
        auto *k = all_owned ? k_sort_count<PT, PT4, true> : k_sort_count<PT, PT4, false>;
        k<<<(n + COUNT_KEYS - 1) / COUNT_KEYS, 256, 0, s>>>(pos, gid, c->keys[0], c->vals[0], (int)n, c->items,
                                                            c->n_items, c->keys[1], (PT4 *)c->spos, c->sgid, c->srow,
                                                            c->sorig, c->cells, c->row2cell);
    } else {
        const bool direct = nb <= SORT_DIRECT_TILES;
        int32_t *offs = direct ? nullptr : c->hist + (int64_t)256 * nb;
        for (int shift = 0; shift < c->key_bits; shift += 8) {
            k_radix_hist<<<nb, SORT_THREADS, 0, s>>>(c->keys[cur], n, shift, c->hist, direct ? 1 : nb, direct ? 256 : 1);
            if (!direct) {
                hipError_t e = vt_launch_scan_i32(c->hist, offs, (int64_t)256 * nb, c->scan_tmp, s);
                if (e != hipSuccess) return e;
            }
            k_radix_scatter<<<nb, SORT_THREADS, 0, s>>>(c->keys[cur], c->vals[cur], c->keys[cur ^ 1], c->vals[cur ^ 1], n,
                                                       shift, c->hist, offs, nb);
            cur ^= 1;
        }
        k_sorted_gather<PT, PT4><<<grid, tpb, 0, s>>>(pos, gid, c->vals[cur], n, c->items, c->n_items, (PT4 *)c->spos,
                                                      c->sgid, c->srow, c->sorig, all_owned, c->cells, c->row2cell);
    }
    c->skey = c->keys[cur];
    // long runs of the table are listed in the spare key buffer (free until the compaction below)
    uint64_t *pieces = c->keys[cur ^ 1];
    const int64_t piece_cap = (n + 1) / 2;
    k_level_table<<<grid, tpb, 0, s>>>(c->skey, n, c->items, c->n_items, c->tab, pieces, piece_cap, c->counters);
    k_level_fill<<<1024, tpb, 0, s>>>(pieces, piece_cap, c->counters, c->tab);
    if (!count && !all_owned) {
        // owned cells in Morton order (flags -> scan -> compact); the flag array reuses vals[cur^1]
        int32_t *flag = (int32_t *)c->vals[cur ^ 1];
        int32_t *scan = (int32_t *)c->keys[cur ^ 1];
        k_owned_flags<<<grid, tpb, 0, s>>>(c->srow, n, flag);
        hipError_t e = vt_launch_scan_i32(flag, scan, n, c->scan_tmp, s);
        if (e != hipSuccess) return e;
        k_owned_compact<<<grid, tpb, 0, s>>>(c->srow, scan, n, c->cells, c->row2cell);
    }
    return hipGetLastError();
}

hipError_t vt_launch_sort(vt_ctx *c, const void *pos, const int32_t *gid) {
    return c->dtype == VT_F32 ? launch_sort<float, float4>(c, (const float *)pos, gid)
                              : launch_sort<double, double4>(c, (const double *)pos, gid);
}
