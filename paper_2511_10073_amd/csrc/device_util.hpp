// Wave64 / workgroup reduction and scan helpers (gfx950: 64-lane wavefronts).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ahr {

constexpr int kWave = 64;

// A pointer into device global memory (address space 1).  Loads through it
// are global loads even where the address was formed as an integer, which
// would otherwise give flat loads that also count against the LDS counter.
template <class T>
using GlobalPtr = const __attribute__((address_space(1))) T*;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / kWave; }

// Lane exchanges without the LDS crossbar (every lane of the wave active).
template <int Ctrl>
__device__ __forceinline__ int dpp(int x) {
    return __builtin_amdgcn_mov_dpp(x, Ctrl, 0xf, 0xf, true);
}
constexpr int kDppPrev = 0x138, kDppNext = 0x130;       // the lane below / above, across the wave (zeros at its ends)

// The values of lanes l and l ^ J as a pair of which one is the caller's own
// (which one is unspecified: for operations that commute).
template <int J>
__device__ __forceinline__ void lane_pair(int x, int& a, int& b) {
    a = x;
    if constexpr (J == 1) {
        b = dpp<0xb1>(x);                               // quad [1, 0, 3, 2]
    } else if constexpr (J == 2) {
        b = dpp<0x4e>(x);                               // quad [2, 3, 0, 1]
    } else if constexpr (J == 4) {
        b = dpp<0x1b>(dpp<0x141>(x));                   // mirrored in 8, then in 4
    } else if constexpr (J == 8) {
        b = dpp<0x128>(x);                              // rotated by 8 in 16
    } else {
        static_assert(J == 16 || J == 32, "lane distance");
        const auto r = J == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                               : __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = static_cast<int>(r[0]);
        b = static_cast<int>(r[1]);
    }
}

// v of lane l plus v of lane l ^ J, for a 64-bit integer or a double.
template <int J, class T>
__device__ __forceinline__ T pair_sum(T v) {
    static_assert(sizeof(T) == 8, "two words");
    struct Words {
        int w[2];
    };
    const Words x = __builtin_bit_cast(Words, v);
    Words a, b;
    lane_pair<J>(x.w[0], a.w[0], b.w[0]);
    lane_pair<J>(x.w[1], a.w[1], b.w[1]);
    return __builtin_bit_cast(T, a) + __builtin_bit_cast(T, b);
}

// Sum over the wave, in every lane (halves first, then quarters, ...).
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
    v = pair_sum<32>(v);
    v = pair_sum<16>(v);
    v = pair_sum<8>(v);
    v = pair_sum<4>(v);
    v = pair_sum<2>(v);
    return pair_sum<1>(v);
}

template <class T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        T u = __shfl_xor(v, o);
        v = u > v ? u : v;
    }
    return v;
}

template <class T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        T u = __shfl_xor(v, o);
        v = u < v ? u : v;
    }
    return v;
}

// v plus the value of the lane that the exchange Ctrl takes it from, in the
// rows of 16 lanes in Rows, where there is one.
template <int Ctrl, int Rows = 0xf>
__device__ __forceinline__ int64_t dpp_add(int64_t v) {
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), Ctrl, Rows, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), Ctrl, Rows, 0xf, false);
    return v + static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32 | static_cast<uint32_t>(lo));
}

// Inclusive scan over each row of 16 lanes: the lanes 1, 2, 4 and 8 below.
__device__ __forceinline__ int64_t row_incl_scan_i64(int64_t v) {
    return dpp_add<0x118>(dpp_add<0x114>(dpp_add<0x112>(dpp_add<0x111>(v))));
}

// Inclusive scan over the wave: the rows, then lane 15 of the row below into
// the odd rows, then lane 31 into the upper two.
__device__ __forceinline__ int64_t wave_incl_scan_i64(int64_t v) {
    return dpp_add<0x143, 0xc>(dpp_add<0x142, 0xa>(row_incl_scan_i64(v)));
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
    return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32 | static_cast<uint32_t>(lo));
}

// From the waves' sums red[w * stride]: the sum of those before the caller's
// wave, and of all (a loop over the 16 waves of a workgroup of 1024 in every
// lane cost the small scans more than all the rest).
template <int BT>
__device__ __forceinline__ void across_waves(const int64_t* red, int stride, int64_t* before, int64_t* total) {
    constexpr int W = BT / kWave;
    static_assert(W <= 16, "waves of a workgroup");
    const int l = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
    const int64_t r = row_incl_scan_i64(l < W ? red[l * stride] : 0);
    *total = readlane_i64(r, W - 1);
    *before = w ? readlane_i64(r, w - 1) : 0;
}

// Block-wide sum; every thread gets the result. red: BT/64 slots.
template <int BT>
__device__ __forceinline__ int64_t block_sum_i64(int64_t v, int64_t* red) {
    v = wave_sum(v);
    __syncthreads();
    if (lane_id() == 0) red[wave_id()] = v;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int w = 0; w < BT / kWave; ++w) t += red[w];
    return t;
}

// Fixed-order block sum of doubles (deterministic for a given block size).
template <int BT>
__device__ __forceinline__ double block_sum_f64(double v, double* red) {
    v = wave_sum(v);
    __syncthreads();
    if (lane_id() == 0) red[wave_id()] = v;
    __syncthreads();
    double t = 0;
#pragma unroll
    for (int w = 0; w < BT / kWave; ++w) t += red[w];
    return t;
}

// The same for W doubles a thread with one pass of the barriers.  red is free
// before the call (a caller that uses it again puts a barrier between).
template <int BT, int W>
__device__ __forceinline__ void block_sums_f64(double (&v)[W], double (*red)[BT / kWave]) {
#pragma unroll
    for (int c = 0; c < W; ++c) {
        const double t = wave_sum(v[c]);
        if (lane_id() == 0) red[c][wave_id()] = t;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < W; ++c) {
        v[c] = 0;
#pragma unroll
        for (int w = 0; w < BT / kWave; ++w) v[c] += red[c][w];
    }
}

// Block exclusive scan of int64; *total gets the block sum. red: BT/64 slots.
template <int BT>
__device__ __forceinline__ int64_t block_exclusive_scan_i64(int64_t v, int64_t* red, int64_t* total) {
    int64_t inc = wave_incl_scan_i64(v);
    __syncthreads();
    if (lane_id() == kWave - 1) red[wave_id()] = inc;
    __syncthreads();
    int64_t before;
    across_waves<BT>(red, 1, &before, total);
    return before + inc - v;
}

// Ordered compaction inside a block: returns the slot of a set flag among
// the set flags of this pass (in thread order) and the pass total.
template <int BT>
__device__ __forceinline__ int block_rank(bool flag, int* red, int* total) {
    uint64_t m = __ballot(flag);
    int l = lane_id();
    uint64_t lt = l ? (~0ull >> (kWave - l)) : 0ull;
    int in_wave = __popcll(m & lt);
    __syncthreads();
    if (l == 0) red[wave_id()] = __popcll(m);
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BT / kWave; ++w) {
        int r = red[w];
        if (w < wave_id()) before += r;
        tot += r;
    }
    *total = tot;
    return before + in_wave;
}

__device__ __forceinline__ float bits_f(int v) { return __int_as_float(v); }
__device__ __forceinline__ int f_bits(float v) { return __float_as_int(v); }

// Workgroups over rows in spatial order are renumbered so that each XCD (blocks
// are dealt round-robin over the 8 XCDs) takes one contiguous range of rows:
// their gathers then share that XCD's L2.
constexpr int kXcds = 8;

// b in [0, nb), nb a multiple of kXcds: a bijection onto [0, nb) that gives
// XCD x (blocks b with b % kXcds == x) the tiles [x nb/8, (x+1) nb/8).
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nb) {
    int64_t per = nb / kXcds;
    return (b % kXcds) * per + b / kXcds;
}

// The least multiple of kXcds not below nb.
inline unsigned xcd_grid(int64_t nb) { return static_cast<unsigned>((nb + kXcds - 1) / kXcds * kXcds); }

}  // namespace ahr
