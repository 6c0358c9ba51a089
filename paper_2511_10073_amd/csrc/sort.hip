// Stable bucket sort of small integer keys (bins, macros, row classes, the
// digits of the layout's keys).  Every position comes from integer counts,
// so the order is exact and the same from run to run.
//
// A workgroup of W waves takes a tile of W x I x 64 consecutive elements,
// each wave one contiguous part of it, and each wave ranks its elements with
// ballots against a counter array of its own in LDS.  The serial chain (a
// counter read and written per 64 elements) is what bounds the scatter, so
// the tile is spread over W waves instead of run through one: 64 elements at
// a time by one wave, 32 times over, took 43 us a sort at 2.2M elements and
// 1,024 keys (24 us at 210,000, and 33 us at 2,000 with 2,048 keys).  The
// larger tiles also make the table of (key, tile) counts an eighth as long,
// so it is written and read in key order without the two transposes.
// Sorting 1,024 keys now takes 17 + 10 + 31 us (count, scan, scatter) at 2.2M
// elements where count, transposes, scan and scatter took 13 + 16 + 20 + 42,
// 4.6 + 7 + 5.7 at 210,000 (5 + 8 + 8 + 25), and 9 at 2,000 (54 in seven
// launches).
#include <algorithm>

#include "ahr_internal.hpp"
#include "device_util.hpp"

namespace ahr {

namespace {

constexpr int kMaxKeys = 16384;
constexpr int kMaxWaves = 8;
constexpr int kMaxIters = 16;
// Counter words of a workgroup: 128 KB of LDS.  Above 4,096 keys that means
// fewer waves; half of it (and half the waves) took 49 against 35 us in the
// scatter of 0.7M elements with 8,000 keys.
constexpr int kLdsWords = 32768;
// Up to kSmallIters x 64 elements a wave one workgroup of up to 16 waves does
// the whole sort, in one launch instead of four.
constexpr int kSmallIters = 16;
constexpr int kSmallStep = 2;
constexpr int kSmallWaves = 16;
// (key, tile) counters above which the keys are sorted in two passes, by halves
// of their bits: every counter is a line written, read by the scan and read
// again.  With 16,384 keys one pass takes 222 us for the counts and 370 for the
// scatter at 2.2M elements, where the former tile-major table with its
// transposes took 415 in all; the hints of that placement are rebuilt in 1672
// us with one pass, 1108 with two, at 1M cells in 1024 and 820.
constexpr int64_t kMaxTable = int64_t(1) << 21;

__device__ __forceinline__ int sort_key(const SortKeys& k, int64_t i) {
    const int v = k.key[i];
    return v < 0 ? -1 : (v >> k.shift) & k.mask;
}

// The elements that may have a key.
__device__ __forceinline__ int32_t sort_count(const SortKeys& k, int32_t n) { return k.count ? *k.count : n; }

__device__ __forceinline__ void wave_lds_order() {
    // LDS serves a wave's accesses in order; the compiler keeps them so
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The 64 keys b of a wave take their places (run[key] = the key's next
// place): returns the lane's place, or -1 without a key.
__device__ __forceinline__ int place_keys(int b, int bits, int32_t* run) {
    const int l = lane_id();
    const uint64_t lt = l ? (~0ull >> (kWave - l)) : 0ull;
    const uint64_t gt = (l == kWave - 1) ? 0ull : (~0ull << (l + 1));
    const bool valid = b >= 0;
    uint64_t peer = __ballot(valid);
    for (int k = 0; k < bits; ++k) {
        const bool bit = valid && ((b >> k) & 1);
        const uint64_t m = __ballot(bit);
        peer &= bit ? m : ~m;
    }
    int at = -1;
    if (valid) at = run[b] + __popcll(peer & lt);
    wave_lds_order();
    if (valid && (peer & gt) == 0) run[b] = at + 1;
    wave_lds_order();
    return at;
}

__device__ __forceinline__ void put(const SortKeys& k, int64_t i, int at, int32_t* list) {
    if (at < 0) return;
    const int32_t v = k.idx ? k.idx[i] : static_cast<int32_t>(i);
    list[at] = v;
    if (k.inverse) k.inverse[v] = at;
    if (k.sorted) k.sorted[at] = k.key[i];
}

// Elements of each key in each tile, key by key: hist[key][tile].
template <int I>
__global__ void __launch_bounds__(kMaxWaves * kWave) k_bucket_count(SortKeys k, int32_t n, int nkeys, int32_t ntiles,
                                                                    int32_t* __restrict__ hist) {
    extern __shared__ int32_t h[];
    const int32_t count = sort_count(k, n);
    for (int b = threadIdx.x; b < nkeys; b += blockDim.x) h[b] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * I * blockDim.x;
    int key[I];       // the tile's keys, all loads in flight together
#pragma unroll
    for (int t = 0; t < I; ++t) {
        const int64_t i = base + static_cast<int64_t>(t) * blockDim.x + threadIdx.x;
        key[t] = sort_key(k, i < n ? i : n - 1);
        if (i >= count) key[t] = -1;
    }
#pragma unroll
    for (int t = 0; t < I; ++t)
        if (key[t] >= 0) atomicAdd(&h[key[t]], 1);
    __syncthreads();
    for (int b = threadIdx.x; b < nkeys; b += blockDim.x)
        hist[static_cast<int64_t>(b) * ntiles + blockIdx.x] = h[b];
}

// Places every element: off[key][tile] (the scanned counts), plus the key's
// count in the tile's earlier waves, plus its rank in its wave.
template <int I>
__global__ void __launch_bounds__(kMaxWaves * kWave) k_bucket_scatter(SortKeys k, int32_t n, int nkeys, int bits,
                                                                      int32_t ntiles, const int32_t* __restrict__ off,
                                                                      int32_t* __restrict__ list,
                                                                      int32_t* __restrict__ start) {
    extern __shared__ int32_t run[];     // [wave][key]
    const int32_t count = sort_count(k, n);
    const int W = blockDim.x / kWave;
    for (int b = threadIdx.x; b < W * nkeys; b += blockDim.x) run[b] = 0;
    __syncthreads();
    int32_t* mine = run + wave_id() * nkeys;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * I * blockDim.x +
                         static_cast<int64_t>(wave_id()) * I * kWave + lane_id();
    int key[I];
#pragma unroll
    for (int t = 0; t < I; ++t) {
        const int64_t i = base + t * kWave;
        key[t] = sort_key(k, i < n ? i : n - 1);
        if (i >= count) key[t] = -1;
    }
#pragma unroll
    for (int t = 0; t < I; ++t)
        if (key[t] >= 0) atomicAdd(&mine[key[t]], 1);
    __syncthreads();
    for (int b = threadIdx.x; b < nkeys; b += blockDim.x) {
        const int first = off[static_cast<int64_t>(b) * ntiles + blockIdx.x];
        if (blockIdx.x == 0) start[b] = first;
        int acc = first;
        for (int w = 0; w < W; ++w) {
            const int c = run[w * nkeys + b];
            run[w * nkeys + b] = acc;
            acc += c;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) start[nkeys] = off[static_cast<int64_t>(nkeys) * ntiles];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < I; ++t) put(k, base + t * kWave, place_keys(key[t], bits, mine), list);
}

// The whole sort by one workgroup: every wave counts and places one
// contiguous part; between the two the counters are scanned key by key,
// waves in order within a key.
__global__ void __launch_bounds__(kSmallWaves * kWave) k_bucket_small(SortKeys k, int32_t n, int nkeys, int bits,
                                                                      int32_t* __restrict__ list,
                                                                      int32_t* __restrict__ start) {
    extern __shared__ int32_t run[];     // [wave][key]
    __shared__ int64_t red[kSmallWaves];
    __shared__ int64_t carry;
    const int32_t count = sort_count(k, n);
    const int W = blockDim.x / kWave;
    for (int b = threadIdx.x; b < W * nkeys; b += blockDim.x) run[b] = 0;
    if (threadIdx.x < kSmallWaves) red[threadIdx.x] = 0;     // (the waves that are not there)
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    int32_t* mine = run + wave_id() * nkeys;
    const int per = (n + static_cast<int>(blockDim.x) - 1) / static_cast<int>(blockDim.x);      // <= kSmallIters
    const int64_t base = static_cast<int64_t>(wave_id()) * per * kWave + lane_id();
    // kSmallStep keys a lane at a time, read again where they are placed: code
    // for all of a lane's keys costs more to fetch than a small input to sort
    int key[kSmallStep];
    const auto load = [&](int t0) {
#pragma unroll
        for (int u = 0; u < kSmallStep; ++u) {
            const int64_t i = base + (t0 + u) * kWave;
            key[u] = sort_key(k, i < n ? i : n - 1);
            if (i >= count || t0 + u >= per) key[u] = -1;
        }
    };
    for (int t0 = 0; t0 < per; t0 += kSmallStep) {
        load(t0);
#pragma unroll
        for (int u = 0; u < kSmallStep; ++u)
            if (key[u] >= 0) atomicAdd(&mine[key[u]], 1);
    }
    __syncthreads();
    for (int b0 = 0; b0 < nkeys; b0 += static_cast<int>(blockDim.x)) {
        const int b = b0 + static_cast<int>(threadIdx.x);
        int64_t c = 0, tot;
        if (b < nkeys)
            for (int w = 0; w < W; ++w) c += run[w * nkeys + b];
        int acc = static_cast<int>(carry + block_exclusive_scan_i64<kSmallWaves * kWave>(c, red, &tot));
        if (b < nkeys) {
            start[b] = acc;
            for (int w = 0; w < W; ++w) {
                const int q = run[w * nkeys + b];
                run[w * nkeys + b] = acc;
                acc += q;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) start[nkeys] = static_cast<int32_t>(carry);
    for (int t0 = 0; t0 < per; t0 += kSmallStep) {
        load(t0);
#pragma unroll
        for (int u = 0; u < kSmallStep; ++u)
            if (t0 + u < per) put(k, base + (t0 + u) * kWave, place_keys(key[u], bits, mine), list);
    }
}

template <int I>
void sort_tiles(const SortKeys& k, int32_t n, int nkeys, int bits, int waves, int32_t* list, int32_t* start,
                DevBuf<int32_t>& i32a, DevBuf<int32_t>& i32b, DevBuf<int64_t>& scan_tmp, hipStream_t s) {
    const int32_t ntiles = static_cast<int32_t>(grid_for(n, I * waves * kWave));
    const int64_t hn = static_cast<int64_t>(nkeys) * ntiles;
    i32a.ensure(static_cast<size_t>(hn) + 1, s);
    i32b.ensure(static_cast<size_t>(hn) + 1, s);
    hipLaunchKernelGGL(k_bucket_count<I>, dim3(ntiles), dim3(waves * kWave), nkeys * sizeof(int32_t), s, k, n, nkeys,
                       ntiles, i32a.p);
    AHR_LAUNCHED("k_bucket_count");
    scan_tmp.ensure(scan_tmp_elems(hn), s);
    scan_i32_to_i32(i32a.p, i32b.p, hn, scan_tmp.p, s);
    hipLaunchKernelGGL(k_bucket_scatter<I>, dim3(ntiles), dim3(waves * kWave),
                       static_cast<size_t>(waves) * nkeys * sizeof(int32_t), s, k, n, nkeys, bits, ntiles, i32b.p, list,
                       start);
    AHR_LAUNCHED("k_bucket_scatter");
}

int key_bits(int nkeys) {
    int bits = 0;
    while ((1 << bits) < nkeys) ++bits;
    return bits;
}

// A tile of the longer form: its waves and the 64-element steps of each.  The
// shortest tile whose (key, tile) table stays within 2^18 counters: short tiles
// give the scatter more waves, but every tile reads and writes its column of
// the table with a line an entry (2.2M elements, 1,024 keys: tiles of 8,192,
// 4,096 and 2,048 take 30, 39 and 74 us in the scatter).
struct Tile {
    int waves, iters;
    int64_t table;       // (key, tile) counters
};

Tile sort_tile(int32_t n, int nkeys) {
    Tile t{std::min(kMaxWaves, kLdsWords / nkeys), 2, 0};
    const auto table = [&]() { return static_cast<int64_t>(nkeys) * grid_for(n, t.iters * t.waves * kWave); };
    while (t.iters < kMaxIters && table() > (1 << 18)) t.iters *= 2;
    t.table = table();
    return t;
}

// One pass (n > 0; list and start hold n and nkeys + 1 entries).
void sort_pass(const SortKeys& k, int32_t n, int nkeys, int32_t* list, int32_t* start, DevBuf<int32_t>& i32a,
               DevBuf<int32_t>& i32b, DevBuf<int64_t>& scan_tmp, hipStream_t s) {
    const int bits = key_bits(nkeys);
    const int small_waves =
        std::min({kSmallWaves, kLdsWords / nkeys, static_cast<int>(std::min(grid_for(n, kWave), 16u))});
    if (n <= small_waves * kSmallIters * kWave) {
        hipLaunchKernelGGL(k_bucket_small, dim3(1), dim3(small_waves * kWave),
                           static_cast<size_t>(small_waves) * nkeys * sizeof(int32_t), s, k, n, nkeys, bits, list, start);
        AHR_LAUNCHED("k_bucket_small");
        return;
    }
    const Tile t = sort_tile(n, nkeys);
    auto f = t.iters == 2   ? sort_tiles<2>
             : t.iters == 4 ? sort_tiles<4>
             : t.iters == 8 ? sort_tiles<8>
                            : sort_tiles<16>;
    f(k, n, nkeys, bits, t.waves, list, start, i32a, i32b, scan_tmp, s);
}

// start[q] = the first place of a key of q or more, from the keys in sorted
// order: a thread a place, and one past the last.
constexpr int kStartBT = 256;
__global__ void __launch_bounds__(kStartBT) k_key_starts(const int32_t* __restrict__ sorted, int shift, int32_t mask,
                                                         const int32_t* __restrict__ count, int nkeys,
                                                         int32_t* __restrict__ start) {
    const int64_t n = *count, p = static_cast<int64_t>(blockIdx.x) * kStartBT + threadIdx.x;
    if (p > n) return;
    const int from = p > 0 ? ((sorted[p - 1] >> shift) & mask) + 1 : 0;
    const int to = p < n ? (sorted[p] >> shift) & mask : nkeys;
    for (int q = from; q <= to; ++q) start[q] = static_cast<int32_t>(p);
}

// The sort in two passes, by the lower and then by the upper half of the key's
// bits.
void sort_halves(const SortKeys& k, int32_t n, int nkeys, int32_t* list, int32_t* start, DevBuf<int32_t>& i32a,
                 DevBuf<int32_t>& i32b, DevBuf<int64_t>& scan_tmp, hipStream_t s) {
    const int lo_bits = key_bits(nkeys) / 2, nlo = 1 << lo_bits, nhi = ((nkeys - 1) >> lo_bits) + 1;
    DevBuf<int32_t> first, keys, sorted, lo_start, hi_start;
    keys.ensure(static_cast<size_t>(n), s);
    SortKeys lo = k;
    lo.mask = k.mask & (nlo - 1);
    lo.inverse = nullptr;
    lo.sorted = keys.p;
    first.ensure(static_cast<size_t>(n), s);
    lo_start.ensure(static_cast<size_t>(nlo) + 1, s);
    sort_pass(lo, n, nlo, first.p, lo_start.p, i32a, i32b, scan_tmp, s);
    SortKeys hi = k;
    hi.key = keys.p;
    hi.idx = first.p;
    hi.count = lo_start.p + nlo;
    hi.shift = k.shift + lo_bits;
    hi.mask = k.mask >> lo_bits;
    if (!hi.sorted) {
        sorted.ensure(static_cast<size_t>(n), s);
        hi.sorted = sorted.p;
    }
    hi_start.ensure(static_cast<size_t>(nhi) + 1, s);
    sort_pass(hi, n, nhi, list, hi_start.p, i32a, i32b, scan_tmp, s);
    hipLaunchKernelGGL(k_key_starts, dim3(grid_for(static_cast<int64_t>(n) + 1, kStartBT)), dim3(kStartBT), 0, s,
                       static_cast<const int32_t*>(hi.sorted), k.shift, k.mask, hi.count, nkeys, start);
    AHR_LAUNCHED("k_key_starts");
    for (auto* b : {&first, &keys, &sorted, &lo_start, &hi_start}) b->release(s);
}

}  // namespace

void bucket_sort(const SortKeys& k, int32_t n, int nkeys, DevBuf<int32_t>& list, DevBuf<int32_t>& start,
                 DevBuf<int32_t>& i32a, DevBuf<int32_t>& i32b, DevBuf<int64_t>& scan_tmp, hipStream_t s) {
    if (nkeys > kMaxKeys) throw Error{AHR_EUNSUPPORTED, "too many buckets (at most 16384 bins or macros)"};
    list.ensure(static_cast<size_t>(n) + 1, s);
    start.ensure(static_cast<size_t>(nkeys) + 1, s);
    if (n == 0) {
        fill_i32(start.p, nkeys + 1, 0, s);
        return;
    }
    if (sort_tile(n, nkeys).table > kMaxTable)
        sort_halves(k, n, nkeys, list.p, start.p, i32a, i32b, scan_tmp, s);
    else
        sort_pass(k, n, nkeys, list.p, start.p, i32a, i32b, scan_tmp, s);
}

void bucket_sort(Graph& g, const SortKeys& k, int32_t n, int nkeys, DevBuf<int32_t>& list, DevBuf<int32_t>& start,
                 hipStream_t s) {
    bucket_sort(k, n, nkeys, list, start, g.i32a, g.i32b, g.scan_tmp, s);
}

}  // namespace ahr
