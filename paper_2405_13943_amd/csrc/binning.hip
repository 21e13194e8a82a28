// Tile binning: turns per-record tile rectangles into per-tile lists of
// record ids ordered by (depth, record).  The paper does not describe tiling
// (its rasterizer is cited, not specified); this is an exact acceleration of
// the per-pixel compositing order (depth, index).
//
//   1. one scan over the records: the visible ones (at least one covered
//      tile) compacted in record order, and each one's first pair
//      (pair_off), the layout the backward's per-pair partials use;
//   2. emit one (tile id, record) pair per covered tile and sort the pairs by
//      tile id (LSD radix, ceil(log2 tiles) bits in one or more passes of at
//      most 8, each staged through LDS so that writes leave in runs);
//   3. per-tile [start, end);
//   4. sort each tile's list by the unique key (depth bits, record) on chip
//      (positive floats order like their bits).
//
// Frames of few records take one launch (k_bin_small), of somewhat more two
// (k_bin_strips, k_bin_tiles) in place of steps 1 to 4.
//
// Every count that depends on the data (visible records V, pairs P) stays on
// the device: kernels read it from the counters and size their loops from
// it, so the whole chain runs without a host round trip.
#include "gs_device.hpp"
#include "gs_internal.hpp"

#include <algorithm>

namespace gs {

constexpr int kScanBlock = 256;
constexpr int kEmitChunk = 1024;                 // pairs per emission chunk
constexpr int kRsBlock = 256;
constexpr int kRsItemsLarge = 16;                // keys per thread and iteration of a radix pass: large
constexpr int kRsItemsSmall = 4;                 // and small sorts (more workgroups)
constexpr uint32_t kRsSmallMax = 1u << 22;       // pair capacity up to which the small form is used
constexpr int kMaxGrid = 1024;

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct BinWs {
    uint32_t* vis;        // visible record ids in record order, [n_records]
    uint32_t* poff;       // first pair of each visible record in that order, [n_records]
    uint32_t* cfirst;     // visible rank holding pair c * kEmitChunk, [capacity / kEmitChunk + 1]
    uint32_t* tkey[2];    // tile keys, [capacity] each
    uint32_t* tval;       // alternate record-id buffer, [capacity]
    uint64_t* key[2];     // sort keys of tile lists longer than one LDS chunk, [capacity] each
    uint32_t* hist;       // radix histograms, [256 * kMaxGrid]
    uint32_t* coltot;     // per-digit totals of one radix pass, [256]
    uint32_t* longq;      // lists longer than one LDS chunk: count, then tile ids, [1 + n_tiles]
    void* part;           // scan partials, [kMaxGrid + 1] x 8 bytes
    size_t bytes;
};

// key[0] overlays the two tile-key buffers and key[1] the alternate values:
// the long-list sort runs after the tile sort and the ranges are done
static BinWs carve(void* base, int64_t n_records, uint64_t capacity, int32_t n_tiles) {
    BinWs w;
    char* p = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { char* q = p ? p + off : nullptr; off += align256(bytes); return q; };
    const size_t nr = size_t(n_records > 0 ? n_records : 1) * 4, nc = size_t(capacity > 0 ? capacity : 1);
    w.vis = reinterpret_cast<uint32_t*>(take(nr));
    w.poff = reinterpret_cast<uint32_t*>(take(nr));
    w.cfirst = reinterpret_cast<uint32_t*>(take((nc / kEmitChunk + 1) * 4));
    char* a = take(nc * 8);
    char* b = take(nc * 8);
    w.key[0] = reinterpret_cast<uint64_t*>(a);
    w.key[1] = reinterpret_cast<uint64_t*>(b);
    w.tkey[0] = reinterpret_cast<uint32_t*>(a);
    w.tkey[1] = a ? reinterpret_cast<uint32_t*>(a + nc * 4) : nullptr;
    w.tval = reinterpret_cast<uint32_t*>(b);
    w.hist = reinterpret_cast<uint32_t*>(take(size_t(256) * kMaxGrid * 4));
    w.coltot = reinterpret_cast<uint32_t*>(take(256 * 4));
    w.longq = reinterpret_cast<uint32_t*>(take((size_t(n_tiles > 0 ? n_tiles : 0) + 1) * 4));
    w.part = take(size_t(kMaxGrid + 1) * 8);
    w.bytes = off;
    return w;
}

size_t bin_workspace_size(int64_t n_records, uint64_t capacity, int32_t n_tiles) {
    return carve(nullptr, n_records, capacity, n_tiles).bytes;
}

// ---------------------------------------------------------------------------
// small helpers

// counters of a frame without records: no visible record, no pair; an
// uncleared overflow still counts the call (its step's update is skipped)
__global__ void k_counters_empty(uint32_t* __restrict__ counters) {
    if (threadIdx.x == 0) {
        counters[GS_CTR_VISIBLE] = 0u;
        counters[GS_CTR_PAIRS] = 0u;
        if (counters[GS_CTR_STATUS] & GS_STATUS_PAIR_OVERFLOW) counters[GS_CTR_OVERFLOWED] += 1u;
    }
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        p[i] = v;
}

// (visible records, pairs): the pair sum saturates at 2^32 - 1, which is
// above every capacity, so an oversized frame is reported, never wrapped
struct VisPairs {
    uint32_t v, p;
};

__device__ inline uint32_t scan_add(uint32_t a, uint32_t b) { return a + b; }
__device__ inline VisPairs scan_add(VisPairs a, VisPairs b) {
    const uint32_t p = a.p + b.p;
    return {a.v + b.v, p < a.p ? 0xffffffffu : p};
}
__device__ inline uint32_t shfl_up_v(uint32_t x, int off) { return __shfl_up(x, off, kWave); }
__device__ inline VisPairs shfl_up_v(VisPairs x, int off) {
    return {__shfl_up(x.v, off, kWave), __shfl_up(x.p, off, kWave)};
}

// exclusive scan of one value per thread over a B-thread block (s_wave
// holds B / kWave values); total = the block's sum.  Only the
// (associative) scan_add is used.
template <int B = kScanBlock, typename T>
__device__ inline T block_excl_scan(T v, T* s_wave, T& total) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    T inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const T t = shfl_up_v(inc, off);
        if (lane >= off) inc = scan_add(t, inc);
    }
    T ex = shfl_up_v(inc, 1);
    if (lane == 0) ex = T{};
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    T before{};
    total = T{};
#pragma unroll
    for (int w = 0; w < B / kWave; w++) {
        const T s = s_wave[w];
        if (w < wave) before = scan_add(before, s);
        total = scan_add(total, s);
    }
    __syncthreads();
    return scan_add(before, ex);
}

// chunk of items [lo, hi) that block b of G handles when n items are split
__device__ inline void block_range(uint32_t n, int G, int b, uint32_t granule, uint32_t& lo, uint32_t& hi) {
    uint32_t chunk = (n + G - 1) / G;
    chunk = (chunk + granule - 1) / granule * granule;
    lo = min(n, uint32_t(b) * chunk);
    hi = min(n, lo + chunk);
}

// ---------------------------------------------------------------------------
// reduce-then-scan over a sequence of n items (two launches: per-block
// sums, then each block's exclusive prefixes)

struct RecordScan {       // item i: record i; output: compacted ids and first pairs
    using T = VisPairs;
    const uint4* meta;
    uint32_t* vis;
    uint32_t* pair_off;       // by record
    uint32_t* poff;           // by visible rank
    uint32_t* cfirst;         // by emission chunk: the visible rank holding its first pair
    uint64_t capacity;
    __device__ T value(uint32_t i) const {
        const uint32_t n = meta_tiles(meta[i].y);
        return {n > 0 ? 1u : 0u, n};
    }
    __device__ void emit(uint32_t i, T pre, T v) const {
        if (v.v) {
            vis[pre.v] = i;
            poff[pre.v] = pre.p;
            pair_off[i] = pre.p;
            // the emission chunks whose first pair is one of this record's
            const uint64_t p0 = pre.p, p1 = min(p0 + v.p, capacity);
            for (uint64_t c = (p0 + kEmitChunk - 1) / kEmitChunk; c * kEmitChunk < p1; c++) cfirst[c] = pre.v;
        }
    }
    __device__ static void finish(T total, uint32_t* counters, uint64_t capacity) {
        counters[GS_CTR_VISIBLE] = total.v;
        counters[GS_CTR_PAIRS] = total.p;
        if (uint64_t(total.p) > capacity) counters[GS_CTR_STATUS] |= GS_STATUS_PAIR_OVERFLOW;
        if (counters[GS_CTR_STATUS] & GS_STATUS_PAIR_OVERFLOW) counters[GS_CTR_OVERFLOWED] += 1u;
    }
};

// The reduce also zeroes `clear[0, n_clear)` (grid-stride) and the word
// `*clear1` (when not null), for buffers the later steps fill in part or
// count into: it saves launches.  kReduceBlock threads per workgroup over
// the ranges of kScanBlock granules.
constexpr int kReduceBlock = 1024;
template <typename F>
__global__ __launch_bounds__(kReduceBlock) void k_scan_reduce(F f, uint32_t n, typename F::T* __restrict__ part,
                                                              int G, uint32_t* __restrict__ clear, int64_t n_clear,
                                                              uint32_t* __restrict__ clear1) {
    using T = typename F::T;
    __shared__ T s_wave[kReduceBlock / kWave];
    for (int64_t i = int64_t(blockIdx.x) * kReduceBlock + threadIdx.x; i < n_clear; i += int64_t(G) * kReduceBlock)
        clear[i] = 0u;
    if (clear1 != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *clear1 = 0u;
    uint32_t lo, hi;
    block_range(n, G, blockIdx.x, kScanBlock, lo, hi);
    T acc{};
    for (uint32_t i = lo + threadIdx.x; i < hi; i += kReduceBlock) acc = scan_add(acc, f.value(i));
    T tot;
    block_excl_scan<kReduceBlock>(acc, s_wave, tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Each workgroup's exclusive prefix is the sum of the partials before it (at
// most kMaxGrid, read by the whole workgroup), then its items' prefixes in
// chunks of kApplyBlock (the reduce's ranges, kApplyBlock threads: fewer
// rounds of the block scan); the last workgroup also hands the total to
// F::finish.
constexpr int kApplyBlock = 1024;
template <typename F>
__global__ __launch_bounds__(kApplyBlock) void k_scan_apply(F f, uint32_t n, const typename F::T* __restrict__ part,
                                                            int G, uint32_t* __restrict__ counters,
                                                            uint64_t capacity) {
    using T = typename F::T;
    __shared__ T s_wave[kApplyBlock / kWave];
    T before{};
    for (int i = threadIdx.x; i < int(blockIdx.x); i += kApplyBlock) before = scan_add(before, part[i]);
    T carry;
    block_excl_scan<kApplyBlock>(before, s_wave, carry);
    if (blockIdx.x == unsigned(G - 1) && threadIdx.x == 0) F::finish(scan_add(carry, part[G - 1]), counters, capacity);
    uint32_t lo, hi;
    block_range(n, G, blockIdx.x, kScanBlock, lo, hi);
    for (uint32_t base = lo; base < hi; base += kApplyBlock) {
        const uint32_t i = base + threadIdx.x;
        const T v = i < hi ? f.value(i) : T{};
        T tot;
        const T ex = block_excl_scan<kApplyBlock>(v, s_wave, tot);
        if (i < hi) f.emit(i, scan_add(carry, ex), v);
        carry = scan_add(carry, tot);
    }
}

// ---------------------------------------------------------------------------
// stable LSD radix sort of (uint32 key, uint32 value) by digits of `bits`
// bits (at most 8), reduce-then-scan with a fixed grid of G workgroups over a
// device-sized n; each workgroup takes a contiguous range of the keys

__device__ __forceinline__ uint32_t digit_of(uint32_t k, int shift, int bits) {
    return (k >> shift) & ((1u << bits) - 1u);
}

__global__ __launch_bounds__(kRsBlock) void k_rs_hist(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ n_dev,
                                                      uint32_t n_host, int shift, int bits, uint32_t* __restrict__ hist,
                                                      int G, uint32_t granule) {
    __shared__ uint32_t h[kRsBlock / kWave][256];
    const int wave = threadIdx.x / kWave;
    for (int i = threadIdx.x; i < 256 * (kRsBlock / kWave); i += kRsBlock) (&h[0][0])[i] = 0;
    __syncthreads();
    const uint32_t n = min(*n_dev, n_host);
    uint32_t lo, hi;
    block_range(n, G, blockIdx.x, granule, lo, hi);
    for (uint32_t i = lo + threadIdx.x; i < hi; i += kRsBlock) atomicAdd(&h[wave][digit_of(keys[i], shift, bits)], 1u);
    __syncthreads();
    const int d = threadIdx.x;
    uint32_t s = 0;
#pragma unroll
    for (int w = 0; w < kRsBlock / kWave; w++) s += h[w][d];
    hist[d * G + blockIdx.x] = s;
}

// one workgroup per digit: exclusive scan of that digit's counts over the G
// workgroups (in place) and the digit's total; the digits' base offsets are
// then an exclusive scan of 256 totals, done by every scatter workgroup
__global__ __launch_bounds__(kRsBlock) void k_rs_colscan(uint32_t* __restrict__ hist, int G,
                                                         uint32_t* __restrict__ coltot) {
    __shared__ uint32_t s_wave[kRsBlock / kWave];
    uint32_t* col = hist + size_t(blockIdx.x) * G;
    constexpr int PER = kMaxGrid / kRsBlock;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int i = threadIdx.x * PER + k;
        v[k] = i < G ? col[i] : 0u;
        sum += v[k];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(sum, s_wave, tot);
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int i = threadIdx.x * PER + k;
        if (i < G) col[i] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) coltot[blockIdx.x] = tot;
}

// Scatter: per iteration kRsBlock * ITEMS keys are ranked by digit (wave ballots for
// the rank among equal digits, LDS counts across waves), staged in LDS in
// digit order, then written out by consecutive threads to consecutive
// addresses of each digit's output run.
template <int ITEMS>
__global__ __launch_bounds__(kRsBlock) void k_rs_scatter(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                         uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                         const uint32_t* __restrict__ n_dev, uint32_t n_host, int shift,
                                                         int bits, const uint32_t* __restrict__ hist, int G,
                                                         const uint32_t* __restrict__ coltot) {
    constexpr int NW = kRsBlock / kWave;
    constexpr int PER_WAVE = kWave * ITEMS;
    constexpr int kRsTile = kRsBlock * ITEMS;
    __shared__ uint32_t run[256];          // next output index of each digit
    __shared__ uint32_t loc[256];          // first staging slot of each digit
    __shared__ uint32_t wcnt[NW][256];     // per wave: count, then first rank, of each digit
    __shared__ uint32_t s_wave[NW];
    __shared__ uint32_t sk[kRsTile], sv[kRsTile];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const uint32_t n = min(*n_dev, n_host);
    uint32_t lo, hi;
    block_range(n, G, blockIdx.x, kRsTile, lo, hi);
    {
        uint32_t tot;
        const uint32_t base = block_excl_scan(coltot[tid], s_wave, tot);
        run[tid] = base + hist[tid * G + blockIdx.x];
    }
    for (uint32_t base = lo; base < hi; base += kRsTile) {
        for (int d = lane; d < 256; d += kWave) wcnt[wave][d] = 0;
        __builtin_amdgcn_wave_barrier();
        uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            const uint32_t i = base + wave * PER_WAVE + k * kWave + lane;
            key[k] = 0; val[k] = 0; rank[k] = 0;
            if (i < hi) {
                key[k] = kin[i];
                val[k] = vin[i];
                const uint32_t dg = digit_of(key[k], shift, bits);
                uint64_t peers = __ballot(1);
                for (int bit = 0; bit < bits; bit++) {
                    const uint64_t m = __ballot((dg >> bit) & 1u);
                    peers &= ((dg >> bit) & 1u) ? m : ~m;
                }
                const uint32_t before = wcnt[wave][dg];
                rank[k] = before + uint32_t(__popcll(peers & lanemask_lt()));
                const int leader = 63 - __clzll(peers);
                if (lane == leader) wcnt[wave][dg] = before + uint32_t(__popcll(peers));
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // thread d: the waves' first ranks of digit d, then the digit's first slot
        uint32_t tot = 0;
        {
            const int d = tid;
#pragma unroll
            for (int w = 0; w < NW; w++) {
                const uint32_t c = wcnt[w][d];
                wcnt[w][d] = tot;
                tot += c;
            }
            uint32_t all;
            loc[d] = block_excl_scan(tot, s_wave, all);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            const uint32_t i = base + wave * PER_WAVE + k * kWave + lane;
            if (i < hi) {
                const uint32_t dg = digit_of(key[k], shift, bits);
                const uint32_t pos = loc[dg] + wcnt[wave][dg] + rank[k];
                sk[pos] = key[k];
                sv[pos] = val[k];
            }
        }
        __syncthreads();
        const uint32_t m = min(uint32_t(kRsTile), hi - base);
        for (uint32_t j = tid; j < m; j += kRsBlock) {
            const uint32_t k = sk[j], dg = digit_of(k, shift, bits);
            const uint32_t o = run[dg] + (j - loc[dg]);
            kout[o] = k;
            vout[o] = sv[j];
        }
        __syncthreads();
        run[tid] += tot;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// pair emission and tile ranges

// Pair-parallel emission: workgroup b of G takes the pairs that block b of
// the first radix pass takes (block_range with the same G and granule), in
// chunks of kEmitChunk; each chunk finds the visible records it spans by
// binary search over their first-pair offsets (staged in LDS), so a
// Gaussian covering thousands of tiles is spread over many threads instead
// of serialising one.  With hist set, the workgroup also counts the first
// radix digit (the low bits0 bits of the tile id) of its pairs and stores
// the counts as that pass's histogram column, which saves the pass its
// counting launch.  A chunk's first and last records come from cfirst
// (written by the record scan) instead of binary searches over all visible
// records.
constexpr int kEmitBlock = 256;

__global__ __launch_bounds__(kEmitBlock) void k_emit(const uint4* __restrict__ meta, const uint32_t* __restrict__ vis,
                                                     const uint32_t* __restrict__ poff,
                                                     const uint32_t* __restrict__ cfirst,
                                                     const uint32_t* __restrict__ counters, gs_frame frame,
                                                     uint64_t capacity, uint32_t* __restrict__ tkey,
                                                     uint32_t* __restrict__ tval, int G, uint32_t granule, int bits0,
                                                     uint32_t* __restrict__ hist) {
    static_assert(kEmitBlock == 256, "one histogram bin per thread");
    __shared__ uint32_t s_off[kEmitChunk + 1];
    __shared__ uint32_t s_rec[kEmitChunk + 1];
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0u;
    const uint32_t mask0 = (1u << bits0) - 1u;
    const uint32_t V = counters[GS_CTR_VISIBLE];
    const uint32_t P = uint32_t(min(uint64_t(counters[GS_CTR_PAIRS]), capacity));
    uint32_t lo_e, hi_e;
    block_range(P, G, blockIdx.x, granule, lo_e, hi_e);
    for (uint32_t e0 = lo_e; e0 < hi_e; e0 += kEmitChunk) {
        const uint32_t e1 = min(hi_e, e0 + kEmitChunk);
        // the ranks holding pairs e0 and e1 (both multiples of kEmitChunk
        // unless e1 = P), at most kEmitChunk + 1 of them: the searches below
        // never pick the last one when its first pair is e1
        const uint32_t lo = cfirst[e0 / kEmitChunk];
        const uint32_t hi = e1 < P ? cfirst[e1 / kEmitChunk] : V - 1;
        const uint32_t n = min(uint32_t(kEmitChunk + 1), hi - lo + 1);
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
            s_off[i] = poff[lo + i];
            s_rec[i] = vis[lo + i];
        }
        __syncthreads();
        for (uint32_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
            uint32_t a = 0, b = n - 1;
            while (a < b) {
                const uint32_t mid = (a + b + 1) >> 1;
                if (s_off[mid] <= e) a = mid; else b = mid - 1;
            }
            const uint32_t r = s_rec[a], k = e - s_off[a];
            const uint4 m = meta[r];
            const int j = job_of_record(frame.jobs, frame.n_jobs, r);
            const uint32_t x0 = m.z & 0xffffu, y0 = m.z >> 16, x1 = m.w & 0xffffu;
            const uint32_t w = x1 - x0 + 1;
            const uint32_t t = uint32_t(frame.jobs[j].tile0) + (y0 + k / w) * uint32_t(frame.jobs[j].tiles_x) + x0 + k % w;
            tkey[e] = t;
            tval[e] = r;
            if (hist != nullptr) atomicAdd(&h[t & mask0], 1u);
        }
        __syncthreads();
    }
    if (hist != nullptr) {
        __syncthreads();
        hist[threadIdx.x * G + blockIdx.x] = h[threadIdx.x];
    }
}

__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ tkey, const uint32_t* __restrict__ counters,
                                                uint64_t capacity, uint2* __restrict__ ranges) {
    const uint32_t P = uint32_t(min(uint64_t(counters[GS_CTR_PAIRS]), capacity));
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < P; e += gridDim.x * blockDim.x) {
        const uint32_t t = tkey[e];
        if (e == 0 || tkey[e - 1] != t) ranges[t].x = e;
        if (e + 1 == P || tkey[e + 1] != t) ranges[t].y = e + 1;
    }
}

// ---------------------------------------------------------------------------
// per-tile depth order: each tile's list (record ids, any order) sorted by the
// unique key (depth bits, record id).
//
// Bucket sort on chip: the depths' bit patterns, scaled linearly over the
// list's own range, pick one of a few buckets per key; LDS atomics count the
// buckets, a scan places them, and each key's place inside its bucket is the
// number of smaller keys there (two or three to compare with on average).
// That is a constant number of LDS round trips per key, where merging sorted
// runs takes one dependent pair per key and round of log2(n / 8) rounds, with
// a binary search each: at lists of 1,300 (the 6M-Gaussian view) 165 -> 84 us
// a launch, at 760 (three 640x417 views of 100k) 41 -> 24.  Depths so clustered
// that a bucket holds more than kBucketMost keys are merge-sorted instead
// (workgroups) or ranked by comparison (wavefronts).
//
// Three forms, by the frame's mean list length (pair capacity / tiles, which
// includes the caller's headroom):
//   kSortWaves  lists of up to 512 by one wavefront each, without a barrier,
//               four to a workgroup, which takes longer ones as a whole.
//               Such lists are bound by the latency of the loads they hang
//               on (range, ids, depths), so what counts is how many are in
//               flight: at a mean of 108 (500k, 1600x1066) every list is, and
//               the launch takes 12 us (19 as a workgroup a list, ranked by
//               comparison; 17 with 256 to a wavefront, as the workgroups
//               with longer lists then go round twice).  At a mean of 220
//               (three served views, 13,660 tiles) 58 -> 36 us;
//   kSortBlocks one list per workgroup of 256: frames whose longer lists would
//               hold up a workgroup of waves, when there are too few tiles to
//               hide it (us, waves / blocks: 1,536 tiles of mean 169 24 / 11,
//               6,767 of 172 28 / 26, 9,126 of 147 21 / 32, 2,752 of 111
//               12 / 12, 6,767 of 65 14 / 19; all bins, 1,080 of 110 54 / 49,
//               of 58 49 / 48, 2,542 of 58 51 / 52, 9,000 of 189 108 / 113, of
//               247 130 / 135, of 329 151 / 147, 14,400 of 193 133 / 155, of
//               295 206 / 228, of 304 212 / 223); short lists by comparison.
//               (Even lists of 115 to 200 in 4,000 to 7,000 tiles would do
//               better as waves, 68 / 73, uneven ones of that mean worse, 92 /
//               79: the capacity does not tell them apart);
//   kSortDense  one list per workgroup of 512, up to 4096 on chip.
// k_tile_sort_long takes the longer lists, one large workgroup each, by
// merging: every thread sorts E consecutive keys in registers (a sorting
// network), then rounds of pairwise merges double the sorted runs; in a round
// each thread produces E consecutive outputs of its pair of runs, finding
// where they start in the two inputs by binary search along the merge path
// and then merging sequentially (ties go to the first run).

constexpr int kSortWaves = 0, kSortBlocks = 1, kSortDense = 2;
constexpr uint64_t kWaveList = 150;                     // mean list length up to which: kSortWaves,
constexpr uint64_t kWaveListMany = 400;                 // and up to which in frames of many tiles
constexpr int64_t kManyTiles = 8192, kFewTiles = 2048;  // below: never kSortWaves
constexpr uint64_t kDenseList = 1024;                   // and above which: kSortDense
constexpr int kSortItems = 8;                           // keys per thread: lists up to 2048 (dense: 4096) on chip
constexpr int kWaveItems = 8;                           // keys per lane of a wavefront's list
constexpr int kWaveMost = kWaveItems * kWave;           // 512
constexpr uint32_t kBucketMost = 32;
constexpr uint32_t kRankMost = 128;                     // a workgroup's lists up to this are ranked by comparison
constexpr int kLongBlock = 1024;
constexpr int kLongItems = 8;
constexpr int kLongChunk = kLongBlock * kLongItems;     // 8192
__host__ __device__ constexpr int sort_block(int form) { return form == kSortDense ? 512 : 256; }
__host__ __device__ constexpr int sort_chunk(int form) { return sort_block(form) * kSortItems; }
__host__ __device__ constexpr int sort_buckets(int form) { return sort_chunk(form) / 2; }

__device__ __forceinline__ uint64_t depth_key(const uint4* __restrict__ meta, uint32_t r) {
    return (uint64_t(meta[r].x) << 32) | r;
}

// number of keys in run[0, n) smaller than k (the run is sorted)
__device__ __forceinline__ uint32_t count_less(const uint64_t* run, uint32_t n, uint64_t k) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (run[mid] < k) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// ascending bitonic network over E keys in registers
template <int E>
__device__ __forceinline__ void sort_registers(uint64_t (&r)[E]) {
#pragma unroll
    for (int k = 2; k <= E; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int i = 0; i < E; i++) {
                const int l = i ^ j;
                if (l > i) {
                    const uint64_t a = r[i], b = r[l];
                    const bool swap = (a > b) == ((i & k) == 0);
                    r[i] = swap ? b : a;
                    r[l] = swap ? a : b;
                }
            }
        }
    }
}

// Sorts sk[0, n) ascending in LDS, n <= B * E, by a workgroup of B threads;
// the keys must be visible to the workgroup (a barrier after they were
// written).  sk must hold ceil(n / E) * E keys (the tail is padded with the
// largest key).  Ends with a barrier.
template <int B, int E>
__device__ void block_merge_sort(uint64_t* sk, uint32_t n) {
    const uint32_t np = (n + E - 1) / E * E;
    const uint32_t base = threadIdx.x * E;
    const bool active = base < np;
    for (uint32_t i = n + threadIdx.x; i < np; i += B) sk[i] = ~0ull;
    __syncthreads();
    uint64_t r[E];
    if (active) {
#pragma unroll
        for (int j = 0; j < E; j++) r[j] = sk[base + j];
        sort_registers<E>(r);
    }
    __syncthreads();
    if (active) {
#pragma unroll
        for (int j = 0; j < E; j++) sk[base + j] = r[j];
    }
    __syncthreads();
    for (uint32_t run = E; run < np; run <<= 1) {
        if (active) {
            const uint32_t a0 = base / (2 * run) * (2 * run);
            const uint32_t a1 = min(a0 + run, np), b1 = min(a0 + 2 * run, np);
            const uint32_t la = a1 - a0, lb = b1 - a1, d = base - a0;
            // outputs [d, d + E) of this pair: how many come from the first run
            uint32_t lo = d > lb ? d - lb : 0u, hi = min(d, la);
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (sk[a0 + mid] <= sk[a1 + d - mid - 1]) lo = mid + 1; else hi = mid;
            }
            uint32_t ia = lo, ib = d - lo;
            uint64_t ka = sk[a0 + min(ia, la - 1)];
            uint64_t kb = lb ? sk[a1 + min(ib, lb - 1)] : 0ull;
#pragma unroll
            for (int j = 0; j < E; j++) {
                const bool from_a = ia < la && (ib >= lb || ka <= kb);
                r[j] = from_a ? ka : kb;
                if (from_a) ia++; else ib++;
                const uint32_t next = from_a ? a0 + min(ia, la - 1) : a1 + min(ib, lb - 1);
                const uint64_t nk = sk[next];
                if (from_a) ka = nk; else kb = nk;
            }
        }
        __syncthreads();
        if (active) {
#pragma unroll
            for (int j = 0; j < E; j++) sk[base + j] = r[j];
        }
        __syncthreads();
    }
}

// Compositing plan for adaptive wavefronts: the tiles grouped by the most
// wavefronts they may take (adaptive_waves of the list length), 4-wave tiles
// first (one workgroup each), then 2-wave, then 1-wave tiles; inside a group
// the longer lists first, by buckets of half the frame's mean list length (the
// last bucket open-ended), so that the heaviest tiles of each group do not
// start last; and the leading share of that list which each pass splits
// (pass_plan).  A counting sort by bin = (group, bucket) over chunks of the
// tiles, in two parts that ride on launches of their own length: workgroups
// of k_tile_sort count each chunk's bins (plan_count), workgroups of
// k_tile_sort_long add the counts up and place their chunk's tiles
// (plan_place).  As one workgroup of 256 beside the sorts the plan kept that
// launch at 20 us at 6,700 tiles (14 without it) and 59 at 13,660 (38).  The
// order inside a bin is whatever the LDS atomics give, which changes no
// result (each tile is composited on its own).
constexpr int kPlanBuckets = 16;
constexpr int kPlanBins = 3 * kPlanBuckets;
constexpr int kPlanBlocks = 1024;           // most chunks
static_assert(kPlanBins <= kWave, "a bin per lane, six bits a bin");
static_assert(kPlanBins * kPlanBlocks <= 256 * kMaxGrid, "the chunks' counts fit the radix histograms' place");

__host__ __device__ inline int plan_blocks(int n_tiles) {
    const int b = (n_tiles + 1023) / 1024;
    return b < kPlanBlocks ? b : kPlanBlocks;
}

struct Plan {
    const uint2* ranges;
    const uint32_t* counters;
    uint32_t* part;             // counts [chunk][kPlanBins]
    uint32_t* order;            // null: no plan
    int n_tiles, quads, blocks;
};

// bin of a tile: group (4, 2, 1 wavefronts) major, then the length bucket,
// longest first.  The bucket is floor(n / (mean / 2)), from a float quotient
// put right in integers
__device__ inline uint32_t plan_bin(const Plan& p, uint32_t pairs, uint2 rg) {
    const uint32_t n = rg.y - rg.x;
    const int w = adaptive_waves(n, pairs, p.n_tiles, p.quads);
    const int grp = w == 4 ? 0 : (w == 2 ? 1 : 2);
    constexpr uint32_t last = kPlanBuckets - 1;
    const uint64_t twice = 2ull * n * uint64_t(p.n_tiles);
    const float half = pairs ? 2.0f * float(p.n_tiles) / float(pairs) : 0.0f;
    uint32_t q = uint32_t(fminf(float(n) * half, float(last)));
    if (q < last && uint64_t(q + 1) * pairs <= twice) q++;
    if (q > 0 && uint64_t(q) * pairs > twice) q--;
    return uint32_t(grp * kPlanBuckets) + last - q;
}

// Adds one to cnt[b] for every active lane and returns the lane's place among
// them: one LDS atomic per distinct b of the wavefront (most tiles share a
// few bins, whose same-address atomics would serialise).
__device__ inline uint32_t plan_slot(uint32_t* cnt, uint32_t b) {
    uint64_t peers = __ballot(1);
    for (int bit = 0; bit < 6; bit++) {
        const uint64_t m = __ballot((b >> bit) & 1u);
        peers &= ((b >> bit) & 1u) ? m : ~m;
    }
    const int leader = __ffsll((long long)peers) - 1;
    uint32_t base = 0u;
    if (lane_id() == leader) base = atomicAdd(&cnt[b], uint32_t(__popcll(peers)));
    base = __shfl(base, leader, kWave);
    return base + uint32_t(__popcll(peers & lanemask_lt()));
}

// tiles of chunk c
__device__ inline void plan_chunk(const Plan& p, int c, int& t0, int& t1) {
    const int per = (p.n_tiles + p.blocks - 1) / p.blocks;
    t0 = min(p.n_tiles, c * per);
    t1 = min(p.n_tiles, t0 + per);
}

// one workgroup: the bins of chunk c counted; cnt: kPlanBins words of LDS
__device__ inline void plan_count(const Plan& p, int c, uint32_t* cnt) {
    if (threadIdx.x < kPlanBins) cnt[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t pairs = p.counters[GS_CTR_PAIRS];
    int t0, t1;
    plan_chunk(p, c, t0, t1);
    for (int t = t0 + int(threadIdx.x); t < t1; t += int(blockDim.x)) plan_slot(cnt, plan_bin(p, pairs, p.ranges[t]));
    __syncthreads();
    if (threadIdx.x < kPlanBins) p.part[c * kPlanBins + int(threadIdx.x)] = cnt[threadIdx.x];
}

// one workgroup (at most 1024 threads): the tiles of chunk c placed; chunk 0
// also writes the counts and shares.  cnt: 2 * kPlanBins words of LDS
__device__ inline void plan_place(const Plan& p, int c, uint32_t* cnt) {
    uint32_t* all = cnt + kPlanBins;
    if (threadIdx.x < 2 * kPlanBins) cnt[threadIdx.x] = 0u;
    __syncthreads();
    const int lane = lane_id(), waves = int(blockDim.x) / kWave;
    uint32_t total = 0u, before = 0u;       // of bin `lane`, over this wavefront's share of the chunks
    if (lane < kPlanBins)
        for (int b = int(threadIdx.x) / kWave; b < p.blocks; b += waves) {
            const uint32_t n = p.part[b * kPlanBins + lane];
            total += n;
            before += b < c ? n : 0u;
        }
    if (lane < kPlanBins) {
        if (total) atomicAdd(&all[lane], total);
        if (before) atomicAdd(&cnt[lane], before);
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        const uint32_t n = lane < kPlanBins ? all[lane] : 0u;
        const uint32_t first = wave_incl_scan_dpp(n) - n;
        if (lane < kPlanBins) cnt[lane] += first;
        if (c == 0) {
            const int bucket = kPlanBuckets - 1 - lane % kPlanBuckets;
            const int bf = min(fwd_split_bucket(p.n_tiles), kPlanBuckets - 1);
            const int bb = min(bwd_split_bucket(p.n_tiles), kPlanBuckets - 1);
            const uint32_t nf = wave_sum_u32(bucket >= bf ? n : 0u), nb = wave_sum_u32(bucket >= bb ? n : 0u);
            const uint32_t n4 = __shfl(first, kPlanBuckets, kWave), n42 = __shfl(first, 2 * kPlanBuckets, kWave);
            if (lane == 0) {
                p.order[0] = n4;
                p.order[1] = n42 - n4;
                p.order[2] = uint32_t(p.n_tiles) - n42;
                // shares in 1/65536, rounded up so that a single tile counts (any
                // share is a valid split: the passes only need the same number)
                const float per = p.n_tiles > 0 ? 65536.0f / float(p.n_tiles) : 0.0f;
                auto share = [&](uint32_t m) { return m > 0 ? min(uint32_t(float(m) * per) + 1u, 0xffffu) : 0u; };
                p.order[3] = share(nf) | share(nb) << 16;
            }
        }
    }
    __syncthreads();
    const uint32_t pairs = p.counters[GS_CTR_PAIRS];
    int t0, t1;
    plan_chunk(p, c, t0, t1);
    for (int t = t0 + int(threadIdx.x); t < t1; t += int(blockDim.x))
        p.order[4 + plan_slot(cnt, plan_bin(p, pairs, p.ranges[t]))] = uint32_t(t);
}

// the plan as launches of its own (frames without the sort's launches)
__global__ __launch_bounds__(1024) void k_tile_plan(Plan p) {
    __shared__ uint32_t cnt[2 * kPlanBins];
    plan_count(p, int(blockIdx.x), cnt);
}
__global__ __launch_bounds__(1024) void k_tile_plan_place(Plan p) {
    __shared__ uint32_t cnt[2 * kPlanBins];
    plan_place(p, int(blockIdx.x), cnt);
}

__device__ inline void wave_lds_order() {    // the wavefront's LDS accesses before against those after
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bucket of depth bits d for a list whose depths span [lo, lo + range]: linear
// over the range, monotone in d, below nb.
struct BucketMap {
    uint32_t lo, mult;     // mult 0: the range is shorter than the buckets, one value each
    __device__ BucketMap(uint32_t lo_, uint32_t range, int nb)
        : lo(lo_), mult(range < uint32_t(nb) ? 0u : uint32_t(float(nb) * 4294967296.0f * 0.9999f / (float(range) + 1.0f))) {}
    __device__ uint32_t operator()(uint32_t d) const { return mult ? __umulhi(d - lo, mult) : d - lo; }
};

// place of key k among the keys [s, e) of its bucket
__device__ __forceinline__ uint32_t bucket_rank(const uint64_t* sk, uint32_t s, uint32_t e, uint64_t k) {
    uint32_t rank = s;
    if (e - s > 1)
        for (uint32_t j = s; j < e; j++) rank += sk[j] < k ? 1u : 0u;
    return rank;
}

// one list of 2 .. kWaveMost entries by one wavefront: sk [kWaveMost] and
// cnt [kWaveMost + 1] are the wavefront's own LDS
__device__ void wave_sort(const uint4* __restrict__ meta, uint32_t* __restrict__ v, uint32_t n, uint64_t* sk,
                          uint32_t* cnt) {
    const uint32_t lane = uint32_t(lane_id());
    uint32_t r[kWaveItems], d[kWaveItems], rank[kWaveItems];
#pragma unroll
    for (int k = 0; k < kWaveItems; k++) {
        const uint32_t i = lane + uint32_t(k) * kWave;
        r[k] = i < n ? v[i] : 0u;
        cnt[i] = 0u;
    }
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int k = 0; k < kWaveItems; k++) {
        const bool in = lane + uint32_t(k) * kWave < n;
        d[k] = in ? meta[r[k]].x : 0u;
        lo = in ? min(lo, d[k]) : lo;
        hi = in ? max(hi, d[k]) : hi;
    }
    lo = wave_min_u32_dpp(lo);
    hi = wave_max_u32_dpp(hi);
    const BucketMap bucket(lo, hi - lo, kWaveMost);
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < kWaveItems; k++)
        if (lane + uint32_t(k) * kWave < n) rank[k] = atomicAdd(&cnt[bucket(d[k])], 1u);
    wave_lds_order();
    // lane: buckets kWaveItems lane .. kWaveItems lane + kWaveItems - 1
    uint32_t c[kWaveItems], sum = 0u, most = 0u;
#pragma unroll
    for (int k = 0; k < kWaveItems; k++) {
        c[k] = cnt[kWaveItems * lane + k];
        sum += c[k];
        most = max(most, c[k]);
    }
    uint32_t run = wave_incl_scan_dpp(sum) - sum;
    most = wave_max_u32_dpp(most);
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < kWaveItems; k++) {
        cnt[kWaveItems * lane + k] = run;
        run += c[k];
    }
    if (lane == kWave - 1) cnt[kWaveMost] = run;
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < kWaveItems; k++)
        if (lane + uint32_t(k) * kWave < n) sk[cnt[bucket(d[k])] + rank[k]] = uint64_t(d[k]) << 32 | r[k];
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < kWaveItems; k++) {
        const uint32_t i = lane + uint32_t(k) * kWave;
        if (i >= n) break;
        const uint64_t key = sk[i];
        const uint32_t b = bucket(uint32_t(key >> 32));
        const bool wide = most > kBucketMost;    // uniform: against all keys
        v[bucket_rank(sk, wide ? 0u : cnt[b], wide ? n : cnt[b + 1], key)] = uint32_t(key);
    }
    wave_lds_order();
}

// one list of 2 .. BLOCK * ITEMS entries by the workgroup: sk [BLOCK * ITEMS],
// cnt [NB + 1], s_tmp [2 * BLOCK / kWave] (all LDS); ends with a barrier
template <int BLOCK, int ITEMS, int NB>
__device__ void block_sort(const uint4* __restrict__ meta, uint32_t* __restrict__ v, uint32_t n, uint64_t* sk,
                           uint32_t* cnt, uint32_t* s_tmp) {
    constexpr int NW = BLOCK / kWave, PER = NB / BLOCK;
    const uint32_t t = threadIdx.x;
    const int wave = int(t / kWave);
    uint32_t r[ITEMS], d[ITEMS], rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        const uint32_t i = t + uint32_t(k) * BLOCK;
        r[k] = i < n ? v[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < PER; k++) cnt[t + uint32_t(k) * BLOCK] = 0u;
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        const bool in = t + uint32_t(k) * BLOCK < n;
        d[k] = in ? meta[r[k]].x : 0u;
        lo = in ? min(lo, d[k]) : lo;
        hi = in ? max(hi, d[k]) : hi;
    }
    lo = wave_min_u32_dpp(lo);
    hi = wave_max_u32_dpp(hi);
    if (lane_id() == 0) {
        s_tmp[wave] = lo;
        s_tmp[NW + wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; w++) {
        lo = min(lo, s_tmp[w]);
        hi = max(hi, s_tmp[NW + w]);
    }
    const BucketMap bucket(lo, hi - lo, NB);
#pragma unroll
    for (int k = 0; k < ITEMS; k++)
        if (t + uint32_t(k) * BLOCK < n) rank[k] = atomicAdd(&cnt[bucket(d[k])], 1u);
    __syncthreads();
    // thread: buckets PER t .. PER t + PER - 1
    uint32_t c[PER], sum = 0u, most = 0u;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        c[k] = cnt[PER * t + k];
        sum += c[k];
        most = max(most, c[k]);
    }
    const uint32_t incl = wave_incl_scan_dpp(sum);
    most = wave_max_u32_dpp(most);
    if (lane_id() == kWave - 1) {
        s_tmp[wave] = incl;
        s_tmp[NW + wave] = most;
    }
    __syncthreads();
    uint32_t run = incl - sum;
#pragma unroll
    for (int w = 0; w < NW; w++) {
        run += w < wave ? s_tmp[w] : 0u;
        most = max(most, s_tmp[NW + w]);
    }
#pragma unroll
    for (int k = 0; k < PER; k++) {
        cnt[PER * t + k] = run;
        run += c[k];
    }
    if (t == BLOCK - 1) cnt[NB] = run;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; k++)
        if (t + uint32_t(k) * BLOCK < n) sk[cnt[bucket(d[k])] + rank[k]] = uint64_t(d[k]) << 32 | r[k];
    __syncthreads();
    if (most > kBucketMost) {          // uniform
        block_merge_sort<BLOCK, ITEMS>(sk, n);
        for (uint32_t i = t; i < n; i += BLOCK) v[i] = uint32_t(sk[i]);
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            const uint32_t i = t + uint32_t(k) * BLOCK;
            if (i >= n) break;
            const uint64_t key = sk[i];
            const uint32_t b = bucket(uint32_t(key >> 32));
            v[bucket_rank(sk, cnt[b], cnt[b + 1], key)] = uint32_t(key);
        }
    }
    __syncthreads();
}

// one list of 2 .. kRankMost entries by the workgroup, each key ranked against
// all: fewer barriers than the buckets; ends with a barrier
__device__ void block_rank(const uint4* __restrict__ meta, uint32_t* __restrict__ v, uint32_t n, uint64_t* sk) {
    const uint32_t i = threadIdx.x;
    const uint64_t k = i < n ? depth_key(meta, v[i]) : 0ull;
    if (i < n) sk[i] = k;
    __syncthreads();
    if (i < n) {
        uint32_t rank = 0u;
        for (uint32_t j = 0; j < n; j++) rank += sk[j] < k ? 1u : 0u;
        v[rank] = uint32_t(k);
    }
    __syncthreads();
}

template <int FORM>
__global__ __launch_bounds__(sort_block(FORM)) void k_tile_sort(const uint4* __restrict__ meta,
                                                                const uint2* __restrict__ ranges, int n_tiles,
                                                                uint32_t* __restrict__ vals,
                                                                uint32_t* __restrict__ longq, Plan plan) {
    constexpr int BLOCK = sort_block(FORM), CHUNK = sort_chunk(FORM), NB = sort_buckets(FORM), NW = BLOCK / kWave;
    __shared__ uint64_t sk[CHUNK];
    __shared__ uint32_t cnt[FORM == kSortWaves ? NW * (kWaveMost + 1) : NB + 1];
    __shared__ uint32_t s_tmp[2 * NW];
    static_assert(FORM != kSortWaves || (NW * kWaveMost <= CHUNK && NB < NW * (kWaveMost + 1)),
                  "the wavefronts' buffers and the workgroup's are the same LDS");
    const int first = plan.order != nullptr ? plan.blocks : 0;
    if (int(blockIdx.x) < first) {          // uniform
        plan_count(plan, int(blockIdx.x), cnt);
        return;
    }
    const int wg = int(blockIdx.x) - first, wgs = int(gridDim.x) - first;
    auto take = [&](int tile, uint2 rg) {       // uniform: a list for the whole workgroup
        const uint32_t n = rg.y - rg.x;
        if (n > uint32_t(CHUNK)) {              // for k_tile_sort_long
            if (threadIdx.x == 0) longq[1 + atomicAdd(&longq[0], 1u)] = uint32_t(tile);
            return;
        }
        if (n <= kRankMost) block_rank(meta, vals + rg.x, n, sk);
        else block_sort<BLOCK, kSortItems, NB>(meta, vals + rg.x, n, sk, cnt, s_tmp);
    };
    if (FORM == kSortWaves) {
        const int wave = int(threadIdx.x / kWave);
        for (int g = wg; g * NW < n_tiles; g += wgs) {
            const int tile = g * NW + wave;
            const uint2 rg = tile < n_tiles ? ranges[tile] : make_uint2(0u, 0u);
            const uint32_t n = rg.y - rg.x;
            if (n >= 2 && n <= uint32_t(kWaveMost))
                wave_sort(meta, vals + rg.x, n, sk + wave * kWaveMost, cnt + wave * (kWaveMost + 1));
            if (__syncthreads_or(n > uint32_t(kWaveMost))) {
                for (int w = 0; w < NW && g * NW + w < n_tiles; w++) {
                    const uint2 rw = ranges[g * NW + w];
                    if (rw.y - rw.x > uint32_t(kWaveMost)) take(g * NW + w, rw);
                }
            }
        }
    } else {
        for (int tile = wg; tile < n_tiles; tile += wgs) {
            const uint2 rg = ranges[tile];
            if (rg.y - rg.x >= 2) take(tile, rg);
        }
    }
}

// Lists longer than k_tile_sort takes (queued by it, in any order): one
// workgroup of kLongBlock threads per list; lists of one chunk of kLongChunk
// keys by buckets, longer ones as chunks merge-sorted in LDS, then pairwise
// merges of sorted runs through two scratch ranges (each key's place is its
// index in its run plus the number of smaller keys in the other run, by
// binary search).
__global__ __launch_bounds__(kLongBlock) void k_tile_sort_long(const uint4* __restrict__ meta,
                                                               const uint2* __restrict__ ranges,
                                                               const uint32_t* __restrict__ longq,
                                                               uint32_t* __restrict__ vals, uint64_t* __restrict__ ka,
                                                               uint64_t* __restrict__ kb, Plan plan) {
    __shared__ uint64_t sk[kLongChunk];
    __shared__ uint32_t cnt[kLongChunk / 2 + 1];
    __shared__ uint32_t s_tmp[2 * kLongBlock / kWave];
    const uint32_t first = plan.order != nullptr ? uint32_t(plan.blocks) : 0u;
    if (blockIdx.x < first) {               // uniform
        plan_place(plan, int(blockIdx.x), cnt);
        return;
    }
    const uint32_t nq = longq[0];
    for (uint32_t q = blockIdx.x - first; q < nq; q += gridDim.x - first) {
        const uint2 rg = ranges[longq[1 + q]];
        const uint32_t n = rg.y - rg.x;
        uint32_t* v = vals + rg.x;
        if (n <= uint32_t(kLongChunk)) {
            block_sort<kLongBlock, kLongItems, kLongChunk / 2>(meta, v, n, sk, cnt, s_tmp);
            continue;
        }
        uint64_t* src = ka + rg.x;
        uint64_t* dst = kb + rg.x;
        for (uint32_t c0 = 0; c0 < n; c0 += kLongChunk) {
            const uint32_t m = min(uint32_t(kLongChunk), n - c0);
            for (uint32_t i = threadIdx.x; i < m; i += kLongBlock) sk[i] = depth_key(meta, v[c0 + i]);
            __syncthreads();
            block_merge_sort<kLongBlock, kLongItems>(sk, m);
            for (uint32_t i = threadIdx.x; i < m; i += kLongBlock) src[c0 + i] = sk[i];
            __syncthreads();
        }
        for (uint32_t run = kLongChunk; run < n; run <<= 1) {
            for (uint32_t i = threadIdx.x; i < n; i += kLongBlock) {
                const uint32_t a0 = (i / (2 * run)) * (2 * run), b0 = a0 + run, b1 = min(a0 + 2 * run, n);
                const uint64_t k = src[i];
                if (b0 >= n) { dst[i] = k; continue; }
                if (i < b0) dst[i + count_less(src + b0, b1 - b0, k)] = k;
                else dst[a0 + (i - b0) + count_less(src + a0, run, k)] = k;
            }
            __syncthreads();
            uint64_t* t = src;
            src = dst;
            dst = t;
        }
        for (uint32_t i = threadIdx.x; i < n; i += kLongBlock) v[i] = uint32_t(src[i]);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// small frames: one launch.  Every tile's workgroup reads the metadata of all
// records, collects those that cover its tile in LDS, sorts them by (depth
// bits, record) and writes the list; where the list starts needs no other
// workgroup, because how many pairs lie in earlier tiles follows in closed
// form from each record's rectangle.  Further workgroups of the launch write
// the records' first pairs and the counters.  The pipeline above takes 8 to 11
// launches of 3 to 8 us each for such frames, all of them waiting.

constexpr int kSmallList = 2048, kSmallListWide = 8192;   // most records of a job (and entries of a list) per form
constexpr int64_t kSmallWork = 12 << 20, kSmallWorkWide = 4 << 20;     // most tiles x records
constexpr int64_t kSmallRecords = 49152;                               // most records of all jobs

// pairs of a record (rectangle m.z, m.w of tiles) in tiles before (c0, ty);
// inside: it has some in tiles c0 to c1 of rows ty to ty1
__device__ __forceinline__ uint32_t pairs_before(const uint4& m, uint32_t c0, uint32_t c1, uint32_t ty, uint32_t ty1,
                                                 bool& inside) {
    const uint32_t x0 = m.z & 0xffffu, y0 = m.z >> 16, x1 = m.w & 0xffffu, y1 = m.w >> 16;
    const uint32_t w = x1 - x0 + 1u;
    inside = c1 >= x0 && c0 <= x1 && ty1 >= y0 && ty <= y1;
    if (ty < y0) return 0u;
    if (ty > y1) return w * (y1 - y0 + 1u);
    return w * (ty - y0) + (c0 > x0 ? min(c0 - x0, w) : 0u);
}

template <int BLOCK>
__device__ inline uint32_t block_sum_u32(uint32_t v, uint32_t* s_wave) {
    v = wave_sum_u32(v);
    __syncthreads();
    if (lane_id() == 0) s_wave[threadIdx.x / kWave] = v;
    __syncthreads();
    uint32_t t = 0u;
#pragma unroll
    for (int w = 0; w < BLOCK / kWave; w++) t += s_wave[w];
    return t;
}

// one workgroup: first pairs of records [4 BLOCK b, 4 BLOCK (b + 1)), after the
// pairs of all records before; the last one also the counters.  s_vp: BLOCK /
// kWave values of LDS
template <int BLOCK>
__device__ inline void write_first_pairs(const uint4* __restrict__ meta, uint32_t nrec, uint32_t b, uint64_t capacity,
                                         uint32_t* __restrict__ pair_off, uint32_t* __restrict__ counters,
                                         VisPairs* s_vp) {
    const uint32_t t = threadIdx.x, lo = b * 4u * BLOCK, hi = min(nrec, lo + 4u * BLOCK);
    constexpr int kAhead = 8;                    // records loaded before any is used
    VisPairs acc{};
    for (uint32_t i0 = t; i0 < lo; i0 += kAhead * BLOCK) {
        uint32_t y[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; k++) y[k] = meta[i0 + (i0 + uint32_t(k) * BLOCK < lo ? uint32_t(k) * BLOCK : 0u)].y;
#pragma unroll
        for (int k = 0; k < kAhead; k++) {
            const uint32_t n = i0 + uint32_t(k) * BLOCK < lo ? meta_tiles(y[k]) : 0u;
            acc = scan_add(acc, VisPairs{n > 0 ? 1u : 0u, n});
        }
    }
    VisPairs carry, tot, four{};
    block_excl_scan<BLOCK>(acc, s_vp, carry);
    const uint32_t i0 = lo + 4u * t;             // a thread's four records
    uint32_t n[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
        n[k] = i0 + k < hi ? meta_tiles(meta[i0 + k].y) : 0u;
        four = scan_add(four, VisPairs{n[k] > 0 ? 1u : 0u, n[k]});
    }
    uint32_t at = scan_add(carry, block_excl_scan<BLOCK>(four, s_vp, tot)).p;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
        if (n[k] > 0) pair_off[i0 + k] = at;
        at += n[k];
    }
    carry = scan_add(carry, tot);
    if (hi == nrec && t == 0) RecordScan::finish(carry, counters, capacity);
}

// A frame with more pairs than capacity: only the first `capacity`, in record
// order, exist.  One workgroup: collect(m, i) for each of them in tile (tx, ty)
// of the job of records [r0, r1); returns how many lie in tiles before.
template <int BLOCK, typename Collect>
__device__ inline uint32_t collect_truncated(const uint4* __restrict__ meta, uint32_t nrec, uint32_t r0, uint32_t r1,
                                             uint32_t tx, uint32_t ty, uint64_t capacity, uint32_t* s_wave,
                                             Collect collect) {
    const uint32_t cap = uint32_t(capacity);
    uint32_t carry = 0u, before = 0u;
    for (uint32_t base = 0; base < nrec && carry < cap; base += BLOCK) {
        const uint32_t i = base + threadIdx.x;
        const uint4 m = meta[i < nrec ? i : 0u];
        const uint32_t n = i < nrec ? meta_tiles(m.y) : 0u;
        uint32_t tot;
        const uint32_t off = carry + block_excl_scan<BLOCK>(n, s_wave, tot);
        carry += tot;
        const uint32_t left = off < cap ? cap - off : 0u;     // of this record's pairs, how many exist
        if (n > 0u && i < r0) before += min(n, left);
        else if (n > 0u && i < r1) {
            bool inside;
            const uint32_t k = pairs_before(m, tx, tx, ty, ty, inside);
            before += min(k, left);
            if (inside && k < left) collect(m, i);
        }
    }
    return block_sum_u32<BLOCK>(before, s_wave);
}

// one workgroup: the n <= CAP keys collected in sk, ordered, to v
template <int BLOCK, int CAP>
__device__ inline void write_sorted(uint64_t* sk, uint32_t n, uint32_t* __restrict__ v) {
    const uint32_t t = threadIdx.x;
    if (n <= uint32_t(BLOCK)) {
        if (t < n) {
            const uint64_t k = sk[t];
            uint32_t rank = 0u;
            for (uint32_t j = 0; j < n; j++) rank += sk[j] < k ? 1u : 0u;
            v[rank] = uint32_t(k);
        }
        return;
    }
    block_merge_sort<BLOCK, CAP / BLOCK>(sk, n);
    for (uint32_t i = t; i < n; i += BLOCK) v[i] = uint32_t(sk[i]);
}

template <int BLOCK, int CAP>
__global__ __launch_bounds__(BLOCK) void k_bin_small(const uint4* __restrict__ meta, gs_frame frame, uint64_t capacity,
                                                     uint32_t* __restrict__ vals, uint2* __restrict__ ranges,
                                                     uint32_t* __restrict__ pair_off, uint32_t* __restrict__ counters) {
    __shared__ uint64_t sk[CAP];
    __shared__ uint32_t s_wave[2 * BLOCK / kWave];
    __shared__ uint32_t s_count;
    const uint32_t nrec = uint32_t(frame.n_records), t = threadIdx.x;
    if (int(blockIdx.x) >= frame.n_tiles) {
        write_first_pairs<BLOCK>(meta, nrec, blockIdx.x - uint32_t(frame.n_tiles), capacity, pair_off, counters,
                                 reinterpret_cast<VisPairs*>(s_wave));
        return;
    }
    const int tile = int(blockIdx.x);
    const gs_job& job = frame.jobs[job_of_tile(frame.jobs, frame.n_jobs, tile)];
    const uint32_t lt = uint32_t(tile - job.tile0);
    const uint32_t tx = lt % uint32_t(job.tiles_x), ty = lt / uint32_t(job.tiles_x);
    const uint32_t r0 = uint32_t(job.rec0), r1 = r0 + uint32_t(job.g1 - job.g0);
    if (t == 0) s_count = 0u;
    __syncthreads();
    auto collect = [&](const uint4& m, uint32_t i) {
        const uint32_t at = atomicAdd(&s_count, 1u);
        if (at < uint32_t(CAP)) sk[at] = uint64_t(m.x) << 32 | i;     // always: a job has at most CAP records
    };
    uint32_t before = 0u, total = 0u;
    constexpr int kAhead = 4;                    // records loaded before any is used
    for (uint32_t i0 = t; i0 < nrec; i0 += kAhead * BLOCK) {
        uint4 m[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; k++) {
            const uint32_t i = i0 + uint32_t(k) * BLOCK;
            m[k] = meta[i < nrec ? i : i0];
        }
#pragma unroll
        for (int k = 0; k < kAhead; k++) {
            const uint32_t i = i0 + uint32_t(k) * BLOCK;
            const uint32_t n = i < nrec ? meta_tiles(m[k].y) : 0u;
            if (n == 0u) continue;
            total += n;
            if (i < r0) before += n;
            else if (i < r1) {
                bool inside;
                before += pairs_before(m[k], tx, tx, ty, ty, inside);
                if (inside) collect(m[k], i);
            }
        }
    }
    total = block_sum_u32<BLOCK>(total, s_wave);
    before = block_sum_u32<BLOCK>(before, s_wave);      // its barriers: every key is collected
    if (uint64_t(total) > capacity) {
        __syncthreads();
        if (t == 0) s_count = 0u;
        __syncthreads();
        before = collect_truncated<BLOCK>(meta, nrec, r0, r1, tx, ty, capacity, s_wave, collect);
    }
    const uint32_t n = min(s_count, uint32_t(CAP));
    if (t == 0) ranges[tile] = n ? make_uint2(before, before + n) : make_uint2(0u, 0u);
    write_sorted<BLOCK, CAP>(sk, n, vals + before);
}

// Frames of somewhat more records: the same in two launches.  k_bin_strips: a
// workgroup reads all records for a strip (`wide` tiles of one row, or the whole
// rows of a narrow view that `wide` tiles hold) and leaves those that meet it
// (key and rectangle) in a list that starts where the strip's pairs will, in
// closed form again; the list is no longer than they are.  (Cut by rows alone,
// narrow or many views had too many strips, us a call by rows / so: 4 views of
// 16k records, 8 x 400 tiles, 1,600 / 392 strips, 114 / 46; 128 views of 500
// records, 16 x 16 tiles, 2,048 / 256 strips, 195 / 74.)
// k_bin_tiles: each tile's workgroup reads its strip's list instead of all
// records; a list too long for its LDS is left for k_tile_sort_long.  All of
// it waits on loads and launches; strips are cut so that a little less than
// one workgroup a CU reads the records (a frame of 20k records, 1,900 tiles:
// 39 us with 512 strips, 33 with 192 or 128; 65k, 6,700 tiles: 112, 92, 96).
// The records' first pairs are written by workgroups ahead of k_bin_tiles',
// beside which they finish: ahead of the strips they were that launch's last
// (33 -> 31 us; 13k records in each of two views of 1,900 tiles 36 -> 31; but
// 20k in each of two of 8,160, where the tiles are the time, 75 -> 78).
// All bins of the first took 53 us in the pipeline's 11 launches, 31 here in 4.
constexpr int kStripBlock = 1024, kStripHold = 4096;        // threads; longest list collected in LDS
constexpr int64_t kStrips = 192;                            // about as many strips
constexpr int64_t kStripRecords = 65536, kStripTiles = 32768;   // most records and tiles
static_assert(kStripRecords * kStripTiles < (int64_t(1) << 32), "sums of pairs fit 32 bits");

// for each tile: its strip's list and its place in the strip
struct StripInfo {
    uint32_t first, count;      // the list; first also: pairs in tiles before the strip
    uint32_t place;             // column | row << 16
    uint32_t overflow;          // the frame has more pairs than capacity: no lists
};

// the strip of a view's tiles: columns [c0, c1], rows [y0, y1]
struct Strip {
    uint32_t c0, c1, y0, y1;
};
static_assert((kStripTiles + kStrips - 1) / kStrips < 256, "a strip's rectangles fit four bytes");
// a / b for a below 2^20 and b > 0: the quotient of a + 1/2 keeps 1 / 2b from
// any whole number, the reciprocal's and the product's rounding less
__device__ __forceinline__ int small_div(int a, int b) {
    return int((float(a) + 0.5f) * __builtin_amdgcn_rcpf(float(b)));
}

// strips of a view: at most two for every `wide` tiles, and one more
struct StripGrid {
    int per_row, rows, strips;      // strips across the view, rows of a strip, strips in all
    __device__ StripGrid(const gs_job& job, int wide)
        : per_row(small_div(job.tiles_x + wide - 1, wide)), rows(max(1, small_div(wide, job.tiles_x))),
          strips(small_div(job.tiles_y + rows - 1, rows) * per_row) {}
};

// Strip i of the frame, the jobs' strips one after the other (wavefront-uniform;
// false past the last).  More than two jobs are counted a lane each: one after
// the other they took half a microsecond apiece.
__device__ inline bool find_strip(const gs_frame& frame, int wide, int i, int& job, Strip& s) {
    job = 0;
    if (frame.n_jobs <= 2) {
        if (frame.n_jobs == 2) {
            const int first = StripGrid(frame.jobs[0], wide).strips;
            job = i >= first ? 1 : 0;
            i -= job ? first : 0;
        }
    } else {
        int before = 0;
        for (int j0 = 0;; j0 += kWave) {
            if (j0 >= frame.n_jobs) return false;
            const int j = j0 + lane_id();
            const int strips = j < frame.n_jobs ? StripGrid(frame.jobs[j], wide).strips : 0;
            const int end = before + int(wave_incl_scan_dpp(uint32_t(strips)));
            const uint64_t after = __ballot(end > i);
            if (after) {
                const int l = __ffsll((long long)after) - 1;
                job = j0 + l;
                i -= __builtin_amdgcn_readlane(end - strips, l);
                break;
            }
            before = __builtin_amdgcn_readlane(end, kWave - 1);
        }
    }
    const gs_job& v = frame.jobs[job];
    const StripGrid g(v, wide);
    if (i >= g.strips) return false;
    const int row = small_div(i, g.per_row);
    s.c0 = uint32_t((i - row * g.per_row) * wide);
    s.c1 = min(s.c0 + uint32_t(wide), uint32_t(v.tiles_x)) - 1u;
    s.y0 = uint32_t(row * g.rows);
    s.y1 = min(s.y0 + uint32_t(g.rows), uint32_t(v.tiles_y)) - 1u;
    return true;
}

// a record's rectangle inside the strip: first column, columns, first row, rows, from the strip's corner
__device__ __forceinline__ uint32_t strip_rect(const uint4& m, const Strip& s) {
    const uint32_t x0 = max(m.z & 0xffffu, s.c0), x1 = min(m.w & 0xffffu, s.c1);
    const uint32_t y0 = max(m.z >> 16, s.y0), y1 = min(m.w >> 16, s.y1);
    return (x0 - s.c0) | (x1 - x0 + 1u) << 8 | (y0 - s.y0) << 16 | (y1 - y0 + 1u) << 24;
}

__global__ __launch_bounds__(kStripBlock, 8) void k_bin_strips(const uint4* __restrict__ meta, gs_frame frame,
                                                            uint64_t capacity, uint64_t* __restrict__ key,
                                                            uint32_t* __restrict__ rect, StripInfo* __restrict__ info,
                                                            int wide, uint32_t* __restrict__ longq) {
    __shared__ uint64_t s_key[kStripHold];
    __shared__ uint32_t s_rect[kStripHold];
    __shared__ uint32_t s_wave[2 * kStripBlock / kWave];
    __shared__ uint32_t s_count;
    const uint32_t nrec = uint32_t(frame.n_records), t = threadIdx.x;
    if (blockIdx.x == 0 && t == 0) *longq = 0u;
    int j;
    Strip st;
    if (!find_strip(frame, wide, int(blockIdx.x), j, st)) return;   // uniform
    const gs_job& job = frame.jobs[j];
    const uint32_t r0 = uint32_t(job.rec0), r1 = r0 + uint32_t(job.g1 - job.g0);
    uint32_t before = 0u, total = 0u;
    if (t == 0) s_count = 0u;
    __syncthreads();
    auto read = [&](uint32_t y1) {      // st.y1; the same as st.y0 for most frames' strips, which saves tests
        constexpr int kAhead = 4;
        for (uint32_t i0 = t; i0 < nrec; i0 += kAhead * kStripBlock) {
            uint4 m[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; k++) {
                const uint32_t i = i0 + uint32_t(k) * kStripBlock;
                m[k] = meta[i < nrec ? i : i0];
            }
#pragma unroll
            for (int k = 0; k < kAhead; k++) {
                const uint32_t i = i0 + uint32_t(k) * kStripBlock;
                const uint32_t n = i < nrec ? meta_tiles(m[k].y) : 0u;
                if (n == 0u) continue;
                total += n;
                if (i < r0) before += n;
                else if (i < r1) {
                    bool inside;
                    before += pairs_before(m[k], st.c0, st.c1, st.y0, y1, inside);
                    if (inside) {
                        const uint32_t at = atomicAdd(&s_count, 1u);
                        if (at < uint32_t(kStripHold)) {
                            s_key[at] = uint64_t(m[k].x) << 32 | i;
                            s_rect[at] = strip_rect(m[k], st);
                        }
                    }
                }
            }
        }
    };
    if (st.y0 == st.y1) read(st.y0);    // uniform
    else read(st.y1);
    total = block_sum_u32<kStripBlock>(total, s_wave);
    before = block_sum_u32<kStripBlock>(before, s_wave);    // its barriers: every record is collected
    const uint32_t count = s_count;
    const bool overflow = uint64_t(total) > capacity;       // uniform
    if (!overflow && count <= uint32_t(kStripHold)) {
        for (uint32_t i = t; i < count; i += kStripBlock) {
            key[before + i] = s_key[i];
            rect[before + i] = s_rect[i];
        }
    } else if (!overflow) {                                 // longer than the LDS holds: another pass
        __syncthreads();
        if (t == 0) s_count = 0u;
        __syncthreads();
        for (uint32_t i = r0 + t; i < r1; i += kStripBlock) {
            const uint4 m = meta[i];
            bool inside = false;
            if (meta_tiles(m.y) > 0u) pairs_before(m, st.c0, st.c1, st.y0, st.y1, inside);
            if (inside) {
                const uint32_t at = before + atomicAdd(&s_count, 1u);
                key[at] = uint64_t(m.x) << 32 | i;
                rect[at] = strip_rect(m, st);
            }
        }
    }
    const uint32_t w = st.c1 - st.c0 + 1u;
    for (uint32_t i = t; i < w * (st.y1 - st.y0 + 1u); i += kStripBlock) {
        const uint32_t y = uint32_t(small_div(int(i), int(w))), x = i - y * w;
        info[job.tile0 + int(st.y0 + y) * job.tiles_x + int(st.c0 + x)] = {before, count, x | y << 16,
                                                                           overflow ? 1u : 0u};
    }
}

constexpr int kBinTileBlock = 256, kBinTileList = 2048;
__global__ __launch_bounds__(kBinTileBlock) void k_bin_tiles(const uint4* __restrict__ meta, gs_frame frame,
                                                             uint64_t capacity, const uint64_t* __restrict__ key,
                                                             const uint32_t* __restrict__ rect,
                                                             const StripInfo* __restrict__ info,
                                                             uint32_t* __restrict__ vals, uint2* __restrict__ ranges,
                                                             uint32_t* __restrict__ longq, int first_wgs,
                                                             uint32_t* __restrict__ pair_off,
                                                             uint32_t* __restrict__ counters) {
    constexpr int BLOCK = kBinTileBlock, CAP = kBinTileList;
    __shared__ uint64_t sk[CAP];
    __shared__ uint32_t s_wave[2 * BLOCK / kWave];
    __shared__ uint32_t s_count;
    const uint32_t t = threadIdx.x;
    if (int(blockIdx.x) < first_wgs) {
        write_first_pairs<BLOCK>(meta, uint32_t(frame.n_records), blockIdx.x, capacity, pair_off, counters,
                                 reinterpret_cast<VisPairs*>(s_wave));
        return;
    }
    const int tile = int(blockIdx.x) - first_wgs;
    const gs_job& job = frame.jobs[job_of_tile(frame.jobs, frame.n_jobs, tile)];
    const uint32_t lt = uint32_t(tile - job.tile0);
    const uint32_t tx = lt % uint32_t(job.tiles_x), ty = lt / uint32_t(job.tiles_x);
    const StripInfo strip = info[tile];
    const uint32_t rx = strip.place & 0xffffu, ry = strip.place >> 16;
    uint32_t before = 0u, n = 0u;
    for (int pass = 0; pass < 2; pass++) {
        // keys to LDS; a list too long for it goes to vals unsorted in a second pass
        if (t == 0) s_count = 0u;
        __syncthreads();
        auto put = [&](uint64_t k) {
            const uint32_t at = atomicAdd(&s_count, 1u);
            if (pass) vals[before + at] = uint32_t(k);
            else if (at < uint32_t(CAP)) sk[at] = k;
        };
        if (strip.overflow) {                             // uniform
            const uint32_t r0 = uint32_t(job.rec0);
            const uint32_t b = collect_truncated<BLOCK>(
                meta, uint32_t(frame.n_records), r0, r0 + uint32_t(job.g1 - job.g0), tx, ty, capacity, s_wave,
                [&](const uint4& m, uint32_t i) { put(uint64_t(m.x) << 32 | i); });
            if (pass == 0) before = b;
        } else {
            uint32_t left = 0u;
            constexpr int kAhead = 4;
            for (uint32_t i0 = t; i0 < strip.count; i0 += kAhead * BLOCK) {
                uint32_t c[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; k++) {
                    const uint32_t i = i0 + uint32_t(k) * BLOCK;
                    c[k] = rect[strip.first + (i < strip.count ? i : i0)];
                }
#pragma unroll
                for (int k = 0; k < kAhead; k++) {
                    const uint32_t i = i0 + uint32_t(k) * BLOCK;
                    const uint32_t x = c[k] & 0xffu, w = c[k] >> 8 & 0xffu, y = c[k] >> 16 & 0xffu, h = c[k] >> 24;
                    if (i >= strip.count) continue;
                    if (ry > y) left += w * min(ry - y, h);
                    if (ry - y >= h) continue;                         // (wraps above y)
                    if (rx > x) left += min(rx - x, w);
                    if (rx - x < w) put(key[strip.first + i]);         // (wraps left of x)
                }
            }
            if (pass == 0) before = strip.first + block_sum_u32<BLOCK>(left, s_wave);
        }
        __syncthreads();
        if (pass) break;
        n = s_count;
        if (t == 0) ranges[tile] = n ? make_uint2(before, before + n) : make_uint2(0u, 0u);
        if (n <= uint32_t(CAP)) {                       // uniform
            write_sorted<BLOCK, CAP>(sk, n, vals + before);
            return;
        }
        __syncthreads();
    }
    if (t == 0) longq[1 + atomicAdd(&longq[0], 1u)] = uint32_t(tile);
}

// ---------------------------------------------------------------------------

static int grid_for(uint64_t n_max, int per_block) {
    uint64_t g = (n_max + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > kMaxGrid) g = kMaxGrid;
    return int(g);
}

// Grid and keys per workgroup of the radix passes over at most n_max keys.
struct RadixShape {
    bool small;
    uint32_t tile;
    int G;
};
static RadixShape radix_shape(uint32_t n_max) {
    const bool small = n_max <= kRsSmallMax;
    const uint32_t tile = kRsBlock * (small ? kRsItemsSmall : kRsItemsLarge);
    return {small, tile, grid_for(n_max, int(tile))};
}
static int radix_passes(int bits) { return (bits + 7) / 8; }
// width of pass p's digit: near-equal widths over the passes
static int radix_digit(int bits, int p) {
    const int passes = radix_passes(bits);
    int shift = 0;
    for (int q = 0; q < p; q++) shift += (bits - shift) / (passes - q);
    return (bits - shift) / (passes - p);
}

// sorts by the low `bits` bits of the keys in passes of at most 8 bits;
// returns (in k_final) the buffer that holds the sorted keys.  With
// first_hist_done the first pass's histogram is already in w.hist (k_emit
// counted it).
static hipError_t radix_sort(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, const uint32_t* n_dev,
                             uint32_t n_max, int bits, bool first_hist_done, uint32_t** k_final, hipStream_t s,
                             BinWs& w) {
    const RadixShape rs = radix_shape(n_max);
    const bool small = rs.small;
    const uint32_t tile = rs.tile;
    const int G = rs.G;
    const int passes = radix_passes(bits);
    uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
    for (int p = 0, shift = 0; p < passes; p++) {
        const int b = radix_digit(bits, p);
        if (p > 0 || !first_hist_done)
            GS_LAUNCH("k_rs_hist", k_rs_hist, dim3(G), dim3(kRsBlock), 0, s, ki, n_dev, n_max, shift, b, w.hist, G,
                      tile);
        GS_LAUNCH("k_rs_colscan", k_rs_colscan, dim3(256), dim3(kRsBlock), 0, s, w.hist, G, w.coltot);
        if (small)
            GS_LAUNCH("k_rs_scatter", k_rs_scatter<kRsItemsSmall>, dim3(G), dim3(kRsBlock), 0, s, ki, vi, ko, vo, n_dev,
                      n_max, shift, b, w.hist, G, w.coltot);
        else
            GS_LAUNCH("k_rs_scatter", k_rs_scatter<kRsItemsLarge>, dim3(G), dim3(kRsBlock), 0, s, ki, vi, ko, vo, n_dev,
                      n_max, shift, b, w.hist, G, w.coltot);
        shift += b;
        uint32_t* t;
        t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    *k_final = ki;
    return hipGetLastError();
}

hipError_t launch_bin_sort(const gs_frame& f, const gs_raster_cfg& cfg, const uint32_t* meta_u32, const gs_bins& bins,
                           void* ws, size_t ws_bytes, hipStream_t s) {
    (void)ws_bytes;
    BinWs w = carve(ws, f.n_records, bins.capacity, f.n_tiles);
    const uint4* meta = reinterpret_cast<const uint4*>(meta_u32);
    const uint32_t nrec = uint32_t(f.n_records);
    uint2* ranges = reinterpret_cast<uint2*>(bins.ranges);
    // counts restart every call (the record scan writes them); the status
    // bits are sticky until the caller clears them
    const int64_t nt = f.n_tiles;
    const bool want_plan = bins.tile_order && (fwd_waves(cfg) == 0 || bwd_waves(cfg) == 0);
    const int quads = (cfg.tile_w / 8) * (cfg.tile_h / 8);
    const Plan plan{ranges, bins.counters, w.hist, want_plan && nt > 0 ? bins.tile_order : nullptr, f.n_tiles, quads,
                    plan_blocks(f.n_tiles)};
    if (nrec == 0) {
        GS_LAUNCH("k_counters_empty", k_counters_empty, dim3(1), dim3(64), 0, s, bins.counters);
        GS_LAUNCH("k_fill_u32", k_fill_u32, dim3(unsigned(std::min<int64_t>((2 * nt + 255) / 256, 2048))), dim3(256), 0,
                  s, bins.ranges, 0u, 2 * nt);
        if (plan.order) {
            GS_LAUNCH("k_tile_plan", k_tile_plan, dim3(unsigned(plan.blocks)), dim3(1024), 0, s, plan);
            GS_LAUNCH("k_tile_plan", k_tile_plan_place, dim3(unsigned(plan.blocks)), dim3(1024), 0, s, plan);
        }
        return hipGetLastError();
    }

    // Frames of few records and tiles: one launch, while a tile's pass over all
    // records costs less than the launches save, and a list fits one
    // workgroup's LDS whatever the records are (a job's are below g_max).  Us
    // a call with the plan, one launch / by strips: 200 records, 16 tiles
    // 8.9 / 15.5; 2k, 1,200 tiles 12.5 / 18.2; 2k, 3,072 tiles 16.8 / 20.8;
    // 2k, 6,700 tiles 24.5 / 24.9; the wide form 8k, 475 tiles 16.0 / 22.4;
    // 5k, 1,200 tiles 22.2 / 20.4; 8k, 1,900 tiles 35.8 / 23.4.  And while one
    // workgroup's walk over the records of all jobs is shorter than the
    // pipeline, one launch / pipeline: 64k in 32 views of 1 tile 48 / 39, in 128
    // 42 / 38, in 8 of 8 tiles 46 / 38; 128k in 64 views of 1 tile 75 / 40.
    const bool wide = f.g_max > kSmallList;
    if (f.g_max <= kSmallListWide && f.n_records <= kSmallRecords && nt > 0 &&
        nt <= (wide ? kSmallWorkWide : kSmallWork) / f.n_records) {
        const int per = 4 * (wide ? 512 : 256);
        const dim3 grid(unsigned(nt + (f.n_records + per - 1) / per));
        if (wide)
            GS_LAUNCH("k_bin_small", (k_bin_small<512, kSmallListWide>), grid, dim3(512), 0, s, meta, f, bins.capacity,
                      bins.vals, ranges, bins.pair_off, bins.counters);
        else
            GS_LAUNCH("k_bin_small", (k_bin_small<256, kSmallList>), grid, dim3(256), 0, s, meta, f, bins.capacity,
                      bins.vals, ranges, bins.pair_off, bins.counters);
        if (plan.order) {
            GS_LAUNCH("k_tile_plan", k_tile_plan, dim3(unsigned(plan.blocks)), dim3(1024), 0, s, plan);
            GS_LAUNCH("k_tile_plan", k_tile_plan_place, dim3(unsigned(plan.blocks)), dim3(1024), 0, s, plan);
        }
        return hipGetLastError();
    }

    // workgroups for the lists k_tile_sort_long may be left: each is longer than `chunk`
    auto long_wgs = [&](uint64_t chunk) {
        return unsigned(std::min<uint64_t>({uint64_t(nt), 256u, bins.capacity / chunk + 1}));
    };
    // By strips while every strip's pass over all records costs less than the
    // pipeline's launches (us a call with the plan, strips / pipeline, one
    // view: 9k records, 64 tiles 28 / 34; 18k, 64 tiles 32 / 36; 40k, 64 tiles
    // 46 / 40; 20k, 256 tiles 33 / 35; 40k, 256 tiles 43 / 38; 60k, 475 tiles
    // 55 / 58; 20k, 1,900 tiles 33 / 53; 65k, 1,900 tiles 61 / 71; 65k, 6,700
    // tiles 92 / 114; 90k, 1,200 tiles 75 / 72; 90k, 6,700 tiles 156 / 134).
    // The number of views makes no difference: 128 of 500 records and 16 tiles
    // each 37 / 50, of 256 tiles 74 / 134.  Of very few tiles, whose lists are
    // then longer than k_bin_tiles sorts, 2,048 records a tile: 16k records, 1
    // tile 180 / 123; 4 tiles 113 / 94; 8 tiles 44 / 80; 16 tiles 35 / 53.
    if (f.n_records <= std::min({kStripRecords, 16384 + 48 * nt, int64_t(kBinTileList) * nt}) && nt <= kStripTiles) {
        static_assert(sizeof(StripInfo) * kStripTiles <= sizeof(uint32_t) * 256 * kMaxGrid, "in the histograms' place");
        StripInfo* info = reinterpret_cast<StripInfo*>(w.hist);
        uint32_t* rect = reinterpret_cast<uint32_t*>(w.key[1]);
        const int per_strip = int((nt + kStrips - 1) / kStrips);
        // a workgroup for every strip: at most two for every per_strip tiles, and one more for a view
        const unsigned strip_wgs = unsigned(std::min<int64_t>(nt, 2 * kStrips + f.n_jobs));
        GS_LAUNCH("k_bin_strips", k_bin_strips, dim3(strip_wgs), dim3(kStripBlock), 0, s, meta, f, bins.capacity,
                  w.key[0], rect, info, per_strip, w.longq);
        const int first_wgs = int((f.n_records + 4 * kBinTileBlock - 1) / (4 * kBinTileBlock));
        GS_LAUNCH("k_bin_tiles", k_bin_tiles, dim3(unsigned(first_wgs + nt)), dim3(kBinTileBlock), 0, s, meta, f,
                  bins.capacity, w.key[0], rect, info, bins.vals, ranges, w.longq, first_wgs, bins.pair_off,
                  bins.counters);
        // the plan's counts take the strips' place
        if (plan.order) GS_LAUNCH("k_tile_plan", k_tile_plan, dim3(unsigned(plan.blocks)), dim3(1024), 0, s, plan);
        GS_LAUNCH("k_tile_sort_long", k_tile_sort_long,
                  dim3((plan.order ? unsigned(plan.blocks) : 0u) + long_wgs(kBinTileList)), dim3(kLongBlock), 0, s,
                  meta, ranges, w.longq, bins.vals, w.key[0], w.key[1], plan);
        return hipGetLastError();
    }

    // 1. visible records in record order, their first pairs; V and P (the
    //    reduce clears the tile ranges, which step 3 fills for tiles with
    //    pairs; and the long-list queue count, which follows the ranges)
    static_assert(sizeof(uint2) == 8, "ranges are pairs of 32-bit words");
    {
        const int G = grid_for(nrec, kScanBlock * 8);
        RecordScan rs{meta, w.vis, bins.pair_off, w.poff, w.cfirst, bins.capacity};
        VisPairs* part = static_cast<VisPairs*>(w.part);
        GS_LAUNCH("k_scan_reduce", k_scan_reduce<RecordScan>, dim3(G), dim3(kReduceBlock), 0, s, rs, nrec, part, G,
                  bins.ranges, 2 * nt, w.longq);
        GS_LAUNCH("k_scan_apply", k_scan_apply<RecordScan>, dim3(G), dim3(kApplyBlock), 0, s, rs, nrec, part, G,
                  bins.counters, bins.capacity);
    }
    // 2. emit (tile, record) pairs in record order, then sort them by tile id
    //    (the emission counts the first radix digit)
    int bits = 0;
    while ((1ll << bits) < nt) bits++;
    const int passes = radix_passes(bits);
    uint32_t* emit_val = (passes & 1) ? w.tval : bins.vals;
    uint32_t* other_val = (passes & 1) ? bins.vals : w.tval;
    const uint32_t pmax = uint32_t(std::min<uint64_t>(bins.capacity, 0xffffffffull));
    if (passes > 0) {
        const RadixShape rs = radix_shape(pmax);
        GS_LAUNCH("k_emit", k_emit, dim3(rs.G), dim3(kEmitBlock), 0, s, meta, w.vis, w.poff, w.cfirst, bins.counters, f,
                  bins.capacity, w.tkey[0], emit_val, rs.G, rs.tile, radix_digit(bits, 0), w.hist);
    } else {
        const int G = grid_for(pmax, kEmitChunk);
        GS_LAUNCH("k_emit", k_emit, dim3(G), dim3(kEmitBlock), 0, s, meta, w.vis, w.poff, w.cfirst, bins.counters, f,
                  bins.capacity, w.tkey[0], emit_val, G, uint32_t(kEmitChunk), 0, static_cast<uint32_t*>(nullptr));
    }
    uint32_t* tk_final = w.tkey[0];
    if (passes > 0) {
        const hipError_t e = radix_sort(w.tkey[0], emit_val, w.tkey[1], other_val, bins.counters + GS_CTR_PAIRS, pmax,
                                        bits, true, &tk_final, s, w);
        if (e != hipSuccess) return e;
    }
    // 3. per-tile [start, end)
    GS_LAUNCH("k_ranges", k_ranges, dim3(2048), dim3(256), 0, s, tk_final, bins.counters, bins.capacity, ranges);
    // 4. each tile's list in (depth bits, record) order, and (5.) beside them
    //    the compositing plan, when a pass splits tiles adaptively
    if (nt > 0) {
        const unsigned plan_wgs = plan.order ? unsigned(plan.blocks) : 0u;
        auto sort = [&](auto kernel, int form, int64_t lists) {
            GS_LAUNCH("k_tile_sort", kernel, dim3(plan_wgs + unsigned(std::min<int64_t>(lists, 4096))),
                      dim3(sort_block(form)), 0, s, meta, ranges, f.n_tiles, bins.vals, w.longq, plan);
        };
        uint64_t chunk = sort_chunk(kSortBlocks);
        if (nt >= kFewTiles && bins.capacity <= uint64_t(nt) * (nt >= kManyTiles ? kWaveListMany : kWaveList))
            sort(k_tile_sort<kSortWaves>, kSortWaves, (nt + 3) / 4);
        else if (bins.capacity <= uint64_t(nt) * kDenseList) sort(k_tile_sort<kSortBlocks>, kSortBlocks, nt);
        else {
            sort(k_tile_sort<kSortDense>, kSortDense, nt);
            chunk = sort_chunk(kSortDense);
        }
        GS_LAUNCH("k_tile_sort_long", k_tile_sort_long, dim3(plan_wgs + long_wgs(chunk)), dim3(kLongBlock), 0, s, meta,
                  ranges, w.longq, bins.vals, w.key[0], w.key[1], plan);
    }
    return hipGetLastError();
}

}  // namespace gs
