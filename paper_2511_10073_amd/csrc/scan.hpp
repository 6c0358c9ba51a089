// Exclusive prefix sums of values that are computed where they are scanned
// and used where they are placed: the flags, counts and class marks of the
// build and of every hint round need no array of their own, and the lists
// made from their ranks no pass of their own.
//
// A job F describes one scan over items 0..n-1 of K int64 sums each (two
// int32 counts below 2^31 can share one):
//   K                                 sums per item
//   kTotal                            item() is given the totals
//   kHeavy                            first() is worth a thread per item
//   Raw first(i)                      item i's values (may also store them)
//   Raw again(i)                      the same, after first(i) ran
//   Pack<K> pack(raw)                 the values as sums; Raw{} for no item
//   void item(i, raw, before, total)  called once per item with its prefix
//   void done(total)                  called once
// Sums are integers, so every result is exact and run-to-run identical.
//
// Up to kScanSmall items one workgroup does it all in one launch (a graph of
// 2,000 cells scans two dozen such arrays; two launches each cost 2.4 + 3.2 us
// and the gap between them, one costs 3).  Longer inputs take two: the tiles'
// sums, then each tile adds up the tiles before it (at most kScanTiles; a few
// KB of cached reads) and scans itself.  A heavy job's first() gets a launch
// of its own before them, with consecutive items in consecutive lanes: the
// 2.7M execution rows took 174 us inside the tile sums, eight items a thread,
// and take 166 that way with the cells' areas and weights formed as well
// (which had a kernel of 147 us).  Up to kScanSmall items it runs inside the one
// launch, unless the job asks for that launch there as well (ahead).
#pragma once

#include "ahr_internal.hpp"
#include "device_util.hpp"

namespace ahr {

template <int K>
struct Pack {
    int64_t v[K];
};

template <int K>
__device__ __forceinline__ void pack_add(Pack<K>& a, const Pack<K>& b) {
#pragma unroll
    for (int k = 0; k < K; ++k) a.v[k] += b.v[k];
}

constexpr int64_t pack2(int64_t lo, int64_t hi) { return lo | (hi << 32); }
__host__ __device__ __forceinline__ int32_t pack_lo(int64_t v) { return static_cast<int32_t>(v & 0xffffffff); }
__host__ __device__ __forceinline__ int32_t pack_hi(int64_t v) { return static_cast<int32_t>(v >> 32); }

constexpr int kScanBT = 256;
// Consecutive items of a thread in a tile: fewer where an item carries many
// sums (8 of four each need 128 registers more than there are).
template <class F>
constexpr int kScanPer = F::K >= 3 ? 2 : 8;
constexpr int kScanSmallBT = 1024;
// Items of a thread at a time in the small form: its cost at a few thousand
// items is fetching its code, which grows with them (2,211 rows: 8.3 us for the
// execution rows with 4, 13.6 with 8; 5.6 and 9.5 for the hint rows), while
// the largest inputs take more rounds of it.
constexpr int kSmallPer = 4;
constexpr int64_t kScanSmall = 16384;
constexpr int64_t kScanTiles = 4096;

// Block exclusive scan of Pack<K>; *total gets the block's sums.
template <int BT, int K>
__device__ __forceinline__ Pack<K> block_scan_pack(Pack<K> v, int64_t (*red)[K], Pack<K>* total) {
    Pack<K> inc = v;
#pragma unroll
    for (int k = 0; k < K; ++k) inc.v[k] = wave_incl_scan_i64(v.v[k]);
    __syncthreads();
    if (lane_id() == kWave - 1)
#pragma unroll
        for (int k = 0; k < K; ++k) red[wave_id()][k] = inc.v[k];
    __syncthreads();
    Pack<K> ex;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int64_t before;
        across_waves<BT>(&red[0][k], K, &before, &total->v[k]);
        ex.v[k] = before + inc.v[k] - v.v[k];
    }
    return ex;
}

// Items base..base+Per-1 of a job (none past n): their values and sums.
template <bool First, int Per, class F>
__device__ __forceinline__ Pack<F::K> scan_load(const F& f, int64_t n, int64_t base, typename F::Raw (&p)[Per]) {
    Pack<F::K> sum{};
#pragma unroll
    for (int k = 0; k < Per; ++k) {
        const int64_t i = base + k < n ? base + k : n - 1;     // clamped: no branch around a load
        if constexpr (First) p[k] = f.first(i);
        else p[k] = f.again(i);
    }
#pragma unroll
    for (int k = 0; k < Per; ++k) {
        if (base + k >= n) p[k] = typename F::Raw{};
        pack_add(sum, f.pack(p[k]));
    }
    return sum;
}

template <int Per, class F>
__device__ __forceinline__ void scan_emit(const F& f, int64_t n, int64_t base, Pack<F::K> run,
                                          const typename F::Raw (&p)[Per], const Pack<F::K>& total) {
#pragma unroll
    for (int k = 0; k < Per; ++k) {
        if (base + k < n) f.item(base + k, p[k], run, total);
        pack_add(run, f.pack(p[k]));
    }
}

template <class F>
struct ScanJob {
    F f;
    int64_t n = 0;
    int64_t tiles = 0;       // 0: nothing to do
    int rounds = 0;          // kScanBT x kScanPer<F> items each, per tile
    int64_t* sums = nullptr; // [tiles][K]
    int ahead = 0;           // a heavy job's first() gets a launch of its own in the small form too
};

// Ahead: first() has run.
template <bool Ahead, class F>
__device__ __forceinline__ void scan_small(const ScanJob<F>& j, int64_t (*red)[F::K]) {
    constexpr int K = F::K;
    constexpr int64_t kStep = static_cast<int64_t>(kScanSmallBT) * kSmallPer;
    typename F::Raw p[kSmallPer];
    Pack<K> carry{}, total{}, tot;
    if constexpr (F::kTotal) {
        for (int64_t b = 0; b < j.n; b += kStep) {
            block_scan_pack<kScanSmallBT, K>(scan_load<!Ahead, kSmallPer>(j.f, j.n, b + threadIdx.x * kSmallPer, p), red, &tot);
            pack_add(total, tot);
        }
    }
    for (int64_t b = 0; b < j.n; b += kStep) {
        const int64_t base = b + threadIdx.x * kSmallPer;
        Pack<K> run = block_scan_pack<kScanSmallBT, K>(scan_load<!F::kTotal && !Ahead, kSmallPer>(j.f, j.n, base, p), red, &tot);
        pack_add(run, carry);
        scan_emit<kSmallPer>(j.f, j.n, base, run, p, total);
        pack_add(carry, tot);
    }
    if (threadIdx.x == 0) j.f.done(carry);
}

// (a heavy job's first() ran in its own launch)
template <class F>
__device__ __forceinline__ void scan_sums(const ScanJob<F>& j, int64_t tile, int64_t (*red)[F::K]) {
    constexpr int K = F::K;
    typename F::Raw p[kScanPer<F>];
    Pack<K> sum{}, tot;
    for (int r = 0; r < j.rounds; ++r) {
        const int64_t base = ((tile * j.rounds + r) * kScanBT + threadIdx.x) * kScanPer<F>;
        pack_add(sum, scan_load<!F::kHeavy, kScanPer<F>>(j.f, j.n, base, p));
    }
    block_scan_pack<kScanBT, K>(sum, red, &tot);
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) j.sums[tile * K + k] = tot.v[k];
}

template <class F>
__device__ __forceinline__ void scan_tile(const ScanJob<F>& j, int64_t tile, int64_t (*red)[F::K]) {
    constexpr int K = F::K;
    constexpr int U = 4;
    Pack<K> pre{}, all{}, tot;
    const int64_t upto = F::kTotal || tile == 0 ? j.tiles : tile;
    for (int64_t b = threadIdx.x; b < upto; b += U * kScanBT) {
        Pack<K> t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = b + u * kScanBT < upto ? b + u * kScanBT : upto - 1;
#pragma unroll
            for (int k = 0; k < K; ++k) t[u].v[k] = j.sums[q * K + k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = b + u * kScanBT;
            if (q < upto) pack_add(all, t[u]);
            if (q < tile) pack_add(pre, t[u]);
        }
    }
    Pack<K> run, total{};
    block_scan_pack<kScanBT, K>(pre, red, &run);
    if (F::kTotal || tile == 0) block_scan_pack<kScanBT, K>(all, red, &total);
    typename F::Raw p[kScanPer<F>];
    for (int r = 0; r < j.rounds; ++r) {
        const int64_t base = ((tile * j.rounds + r) * kScanBT + threadIdx.x) * kScanPer<F>;
        Pack<K> ex = block_scan_pack<kScanBT, K>(scan_load<false, kScanPer<F>>(j.f, j.n, base, p), red, &tot);
        pack_add(ex, run);
        scan_emit<kScanPer<F>>(j.f, j.n, base, ex, p, total);
        pack_add(run, tot);
    }
    if (tile == 0 && threadIdx.x == 0) j.f.done(total);
}

// Up to three jobs side by side: workgroup b takes the first job's tile b,
// then the second's, then the third's (one workgroup a job in the small form).
struct NoScan {
    static constexpr int K = 1;
    static constexpr bool kTotal = false, kHeavy = false;
    using Raw = Pack<1>;
    __device__ Pack<1> first(int64_t) const { return Pack<1>{}; }
    __device__ Pack<1> again(int64_t) const { return Pack<1>{}; }
    __device__ Pack<1> pack(const Pack<1>& p) const { return p; }
    __device__ void item(int64_t, const Pack<1>&, const Pack<1>&, const Pack<1>&) const {}
    __device__ void done(const Pack<1>&) const {}
};

template <bool Ahead, class A, class B, class C>
__global__ void __launch_bounds__(kScanSmallBT) k_scan_small(ScanJob<A> a, ScanJob<B> b, ScanJob<C> c) {
    __shared__ int64_t red[kScanSmallBT / kWave * (A::K > B::K ? (A::K > C::K ? A::K : C::K) : (B::K > C::K ? B::K : C::K))];
    if (blockIdx.x == 0) scan_small<Ahead>(a, reinterpret_cast<int64_t(*)[A::K]>(red));
    else if (blockIdx.x == 1) scan_small<false>(b, reinterpret_cast<int64_t(*)[B::K]>(red));
    else scan_small<false>(c, reinterpret_cast<int64_t(*)[C::K]>(red));
}

template <class A, class B, class C>
__global__ void __launch_bounds__(kScanBT) k_scan_sums(ScanJob<A> a, ScanJob<B> b, ScanJob<C> c) {
    __shared__ int64_t red[kScanBT / kWave * (A::K > B::K ? (A::K > C::K ? A::K : C::K) : (B::K > C::K ? B::K : C::K))];
    const int64_t t = blockIdx.x;
    if (t < a.tiles) scan_sums(a, t, reinterpret_cast<int64_t(*)[A::K]>(red));
    else if (t < a.tiles + b.tiles) scan_sums(b, t - a.tiles, reinterpret_cast<int64_t(*)[B::K]>(red));
    else scan_sums(c, t - a.tiles - b.tiles, reinterpret_cast<int64_t(*)[C::K]>(red));
}

template <class A, class B, class C>
__global__ void __launch_bounds__(kScanBT) k_scan_tiles(ScanJob<A> a, ScanJob<B> b, ScanJob<C> c) {
    __shared__ int64_t red[kScanBT / kWave * (A::K > B::K ? (A::K > C::K ? A::K : C::K) : (B::K > C::K ? B::K : C::K))];
    const int64_t t = blockIdx.x;
    if (t < a.tiles) scan_tile(a, t, reinterpret_cast<int64_t(*)[A::K]>(red));
    else if (t < a.tiles + b.tiles) scan_tile(b, t - a.tiles, reinterpret_cast<int64_t(*)[B::K]>(red));
    else scan_tile(c, t - a.tiles - b.tiles, reinterpret_cast<int64_t(*)[C::K]>(red));
}

template <class F>
__global__ void __launch_bounds__(kScanBT) k_scan_first(ScanJob<F> j) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kScanBT + threadIdx.x;
    if (i < j.n) j.f.first(i);
}

template <class F>
ScanJob<F> scan_job(const F& f, int64_t n) {
    ScanJob<F> j;
    j.f = f;
    j.n = n;
    constexpr int64_t kRound = static_cast<int64_t>(kScanBT) * kScanPer<F>;
    const int64_t r = (n + kRound * kScanTiles - 1) / (kRound * kScanTiles);
    j.rounds = n > 0 ? static_cast<int>(r) : 0;
    // (an empty input still has its done(): one tile of no rounds)
    j.tiles = n > 0 ? (n + kRound * j.rounds - 1) / (kRound * j.rounds) : 1;
    return j;
}

// Runs the jobs on s; tmp is grown as needed.
template <class A, class B = NoScan, class C = NoScan>
void run_scans(ScanJob<A> a, DevBuf<int64_t>& tmp, hipStream_t s, ScanJob<B> b = {}, ScanJob<C> c = {}) {
    if (a.n <= kScanSmall && b.n <= kScanSmall && c.n <= kScanSmall) {
        const unsigned jobs = c.tiles ? 3 : b.tiles ? 2 : 1;
        if constexpr (A::kHeavy) {
            if (a.ahead && a.n > 0) {
                hipLaunchKernelGGL(k_scan_first<A>, dim3(grid_for(a.n, kScanBT)), dim3(kScanBT), 0, s, a);
                AHR_LAUNCHED("k_scan_first");
                hipLaunchKernelGGL((k_scan_small<true, A, B, C>), dim3(jobs), dim3(kScanSmallBT), 0, s, a, b, c);
                AHR_LAUNCHED("k_scan_small");
                return;
            }
        }
        hipLaunchKernelGGL((k_scan_small<false, A, B, C>), dim3(jobs), dim3(kScanSmallBT), 0, s, a, b, c);
        AHR_LAUNCHED("k_scan_small");
        return;
    }
    tmp.ensure(static_cast<size_t>(a.tiles * A::K + b.tiles * B::K + c.tiles * C::K), s);
    a.sums = tmp.p;
    b.sums = a.sums + a.tiles * A::K;
    c.sums = b.sums + b.tiles * B::K;
    static_assert(!B::kHeavy && !C::kHeavy, "only the first job may be heavy");
    if constexpr (A::kHeavy) {
        hipLaunchKernelGGL(k_scan_first<A>, dim3(grid_for(a.n, kScanBT)), dim3(kScanBT), 0, s, a);
        AHR_LAUNCHED("k_scan_first");
    }
    const unsigned blocks = static_cast<unsigned>(a.tiles + b.tiles + c.tiles);
    hipLaunchKernelGGL((k_scan_sums<A, B, C>), dim3(blocks), dim3(kScanBT), 0, s, a, b, c);
    AHR_LAUNCHED("k_scan_sums");
    hipLaunchKernelGGL((k_scan_tiles<A, B, C>), dim3(blocks), dim3(kScanBT), 0, s, a, b, c);
    AHR_LAUNCHED("k_scan_tiles");
}

}  // namespace ahr
