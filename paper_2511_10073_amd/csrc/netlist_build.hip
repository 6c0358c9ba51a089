// Netlist part of the graph: macro pin expansion (Section V, "Macro pin
// expansion") and the clique/star net model with integer weights in units
// of 2^-32, merged into a canonical CSR (rows ascending, columns strictly
// ascending, parallel edges summed exactly).  Every structural step uses
// integer counts, scans and sorts, so the result is bit-identical from run
// to run and to any other exact implementation of the same definition.
#include <algorithm>

#include "ahr_internal.hpp"
#include "device_util.hpp"
#include "scan.hpp"

namespace ahr {

namespace {

constexpr int kBT = 256;

// Device-side validation of the caller's netlist arrays.  bad[0] gets a
// nonzero code on the first violation found.
__global__ void k_validate(const int32_t* __restrict__ net_ptr, int32_t n_nets, const int32_t* __restrict__ pin_node,
                           int32_t n_pins, int32_t n_inst, int32_t* bad) {
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n_pins) {
        int v = pin_node[i];
        if (v < 0 || v >= n_inst) atomicCAS(bad, 0, 1);
    }
    if (i <= n_nets) {
        int a = net_ptr[i];
        if (i == 0 && a != 0) atomicCAS(bad, 0, 2);
        if (i == n_nets && a != n_pins) atomicCAS(bad, 0, 3);
        if (i < n_nets && net_ptr[i + 1] < a) atomicCAS(bad, 0, 4);
    }
}

// The ranks of the pins that become nodes of their own (pins of fixed macros).
struct PinScan {
    static constexpr int K = 1;
    static constexpr bool kTotal = false, kHeavy = false;
    using Raw = Pack<1>;
    __device__ Pack<1> pack(const Pack<1>& p) const { return p; }
    const int32_t* pin_node;
    const uint8_t* flags;
    int32_t n_pins, n_inst, expand;
    uint8_t* is_mp;             // [n_pins] between the passes
    int32_t* rank;              // [n_pins + 1]
    int32_t* count;
    __device__ Pack<1> first(int64_t p) const {
        const int v = pin_node[p];
        const uint8_t f = flags[v >= 0 && v < n_inst ? v : 0];      // clamped: runs before the netlist is verified
        const bool mp = expand && (f & AHR_NODE_FIXED) && (f & AHR_NODE_MACRO);
        is_mp[p] = mp ? 1 : 0;
        return {{mp ? 1 : 0}};
    }
    __device__ Pack<1> again(int64_t p) const { return {{is_mp[p]}}; }
    __device__ void item(int64_t p, const Pack<1>&, const Pack<1>& before, const Pack<1>&) const {
        rank[p] = pack_lo(before.v[0]);
    }
    __device__ void done(const Pack<1>& total) const { rank[n_pins] = *count = pack_lo(total.v[0]); }
};

// Per net: star (more than clique_max pins), big (more pins than a wave),
// big star (a star whose spokes a whole workgroup averages); their ranks.
struct NetScan {
    static constexpr int K = 2;
    static constexpr bool kTotal = false, kHeavy = false;
    using Raw = Pack<2>;
    __device__ Pack<2> pack(const Pack<2>& p) const { return p; }
    const int32_t* net_ptr;
    int32_t n_nets, clique_max;
    int32_t *star, *big, *big_star;      // [n_nets + 1]
    int32_t* counts;                     // the three totals
    __device__ Pack<2> first(int64_t e) const {
        const int deg = net_ptr[e + 1] - net_ptr[e];
        return {{pack2(deg > clique_max ? 1 : 0, deg > kWave ? 1 : 0), deg > clique_max && deg > kStarMid ? 1 : 0}};
    }
    __device__ Pack<2> again(int64_t e) const { return first(e); }
    __device__ void put(int64_t e, const Pack<2>& at) const {
        star[e] = pack_lo(at.v[0]);
        big[e] = pack_hi(at.v[0]);
        big_star[e] = pack_lo(at.v[1]);
    }
    __device__ void item(int64_t e, const Pack<2>&, const Pack<2>& before, const Pack<2>&) const { put(e, before); }
    __device__ void done(const Pack<2>& total) const {
        put(n_nets, total);
        counts[0] = pack_lo(total.v[0]);
        counts[1] = pack_hi(total.v[0]);
        counts[2] = pack_lo(total.v[1]);
    }
};

// The macros' ranks, and the counts of all and of movable macros.
struct MacroScan {
    static constexpr int K = 1;
    static constexpr bool kTotal = false, kHeavy = false;
    using Raw = Pack<1>;
    __device__ Pack<1> pack(const Pack<1>& p) const { return p; }
    const uint8_t* flags;
    int32_t n;
    int32_t* rank;              // [n + 1]
    int32_t* counts;
    __device__ Pack<1> first(int64_t i) const {
        const uint8_t f = flags[i];
        const bool m = f & AHR_NODE_MACRO;
        return {{pack2(m ? 1 : 0, m && !(f & AHR_NODE_FIXED) ? 1 : 0)}};
    }
    __device__ Pack<1> again(int64_t i) const { return first(i); }
    __device__ void item(int64_t i, const Pack<1>&, const Pack<1>& before, const Pack<1>&) const {
        rank[i] = pack_lo(before.v[0]);
    }
    __device__ void done(const Pack<1>& total) const {
        rank[n] = counts[0] = pack_lo(total.v[0]);
        counts[1] = pack_hi(total.v[0]);
    }
};

// What the ranks place, in one launch: the pins' nodes, the lists of macro
// pins, stars, big nets, big stars (by star index) and macros, the net of
// every pin of the nets of at most a wave's worth of pins (k_pin_net_big
// writes the others'), and zeros in the row counters.
struct ListArgs {
    const int32_t *net_ptr, *pin_node;
    int32_t n_pins, n_nets, n_inst;
    const int32_t *mp_rank, *star_rank, *big_rank, *bs_rank, *mac_rank;
    int32_t *pin_node_x, *mp_owner, *mp_pin, *star_net, *big_nets, *big_stars, *macro_ids, *pin_net, *cnt;
    int32_t n_cnt;
};

__global__ void k_build_lists(ListArgs a) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < a.n_cnt) a.cnt[i] = 0;
    if (i < a.n_pins) {
        const int v = a.pin_node[i], r = a.mp_rank[i];
        if (a.mp_rank[i + 1] > r) {
            a.pin_node_x[i] = a.n_inst + r;
            a.mp_owner[r] = v;
            a.mp_pin[r] = static_cast<int32_t>(i);
        } else {
            a.pin_node_x[i] = v;
        }
    }
    if (i < a.n_inst) {
        const int r = a.mac_rank[i];
        if (a.mac_rank[i + 1] > r) a.macro_ids[r] = static_cast<int32_t>(i);
    }
    if (i < a.n_nets) {
        const int e = static_cast<int>(i), s = a.star_rank[i], b = a.big_rank[i], bs = a.bs_rank[i];
        if (a.star_rank[i + 1] > s) a.star_net[s] = e;
        if (a.bs_rank[i + 1] > bs) a.big_stars[bs] = s;
        if (a.big_rank[i + 1] > b) {
            a.big_nets[b] = e;
        } else {
            const int p0 = a.net_ptr[i], p1 = a.net_ptr[i + 1];      // (read once: the stores may alias)
            for (int p = p0; p < p1; ++p) a.pin_net[p] = e;
        }
    }
}

// Net of every pin of the nets with more than a wave's worth of pins, one
// workgroup each.
__global__ void k_pin_net_big(const int32_t* __restrict__ big, const int32_t* __restrict__ net_ptr,
                              int32_t* __restrict__ pin_net) {
    const int e = big[blockIdx.x];
    for (int p = net_ptr[e] + threadIdx.x; p < net_ptr[e + 1]; p += blockDim.x) pin_net[p] = e;
}

// Integer weight of one clique pair / one star spoke (units of 2^-32),
// round-half-even of the float64 value, evaluated in this order:
//   clique: (2^32 w) / (p - 1)     star: ((2^32 w) p) / (p - 1)
__device__ __forceinline__ int64_t q_clique(float w, int p) {
    double wq = static_cast<double>(w) * 4294967296.0;
    return static_cast<int64_t>(__builtin_rint(wq / static_cast<double>(p - 1)));
}
__device__ __forceinline__ int64_t q_star(float w, int p) {
    double wq = static_cast<double>(w) * 4294967296.0;
    double num = wq * static_cast<double>(p);
    return static_cast<int64_t>(__builtin_rint(num / static_cast<double>(p - 1)));
}

// A raw (unsorted, unmerged) entry: column and integer weight, one 16-byte
// store per entry in the scatter and one load in the sorts.
struct alignas(16) RawEnt {
    int32_t col;
    int32_t pad;
    int64_t q;
};

__device__ __forceinline__ RawEnt raw_ent(int32_t col, int64_t q) {
    RawEnt e;
    e.col = col;
    e.pad = 0;
    e.q = q;
    return e;
}

struct NetArgs {
    const int32_t* net_ptr;
    const int32_t* pin_net;
    const int32_t* pin_x;
    const float* net_w;
    const int32_t* star_rank;
    int32_t n_nets, n_pins, clique_max, first_star;
};

// The nodes of the pins of a clique net of at most kNetUnroll pins, all
// loaded at once (indexes clamped to the last pin; a loop one load at a time
// would wait for each), and how many of them differ from v.
constexpr int kNetUnroll = 16;

__device__ __forceinline__ int clique_nodes(const int32_t* __restrict__ pin_x, int lo, int hi, int v, int* node) {
    int c = 0;
    if (hi - lo <= kNetUnroll) {
#pragma unroll
        for (int u = 0; u < kNetUnroll; ++u) node[u] = pin_x[lo + u < hi ? lo + u : hi - 1];
#pragma unroll
        for (int u = 0; u < kNetUnroll; ++u) c += (lo + u < hi && node[u] != v) ? 1 : 0;
    } else {
        for (int b = lo; b < hi; ++b) c += (pin_x[b] != v) ? 1 : 0;
    }
    return c;
}

// Entries each row receives (parallel edges counted separately).  Each pin
// reserves its run of its row's slots here, with the atomic that counts it:
// slot[p] = where the run starts inside the row (the run order inside a row
// does not matter: rows are sorted by column and equal columns merged by
// exact integer sums afterwards).
__global__ void k_row_counts(NetArgs a, int32_t* __restrict__ cnt, int32_t* __restrict__ slot) {
    int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.n_pins) return;
    int e = a.pin_net[p];
    int lo = a.net_ptr[e], hi = a.net_ptr[e + 1];
    int deg = hi - lo;
    if (deg < 2) return;
    int v = a.pin_x[p];
    if (deg <= a.clique_max) {
        int node[kNetUnroll];
        const int c = clique_nodes(a.pin_x, lo, hi, v, node);
        if (c) slot[p] = atomicAdd(&cnt[v], c);
    } else {
        slot[p] = atomicAdd(&cnt[v], 1);
        if (p == lo) cnt[a.first_star + a.star_rank[e]] = deg;
    }
}

// Raw entries: each pin writes its run at the slots it reserved while the
// rows were counted.
__global__ void k_scatter(NetArgs a, const int64_t* __restrict__ rp, const int32_t* __restrict__ slot,
                          RawEnt* __restrict__ raw) {
    int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.n_pins) return;
    int e = a.pin_net[p];
    int lo = a.net_ptr[e], hi = a.net_ptr[e + 1];
    int deg = hi - lo;
    if (deg < 2) return;
    int v = a.pin_x[p];
    float w = a.net_w ? a.net_w[e] : 1.0f;
    if (deg <= a.clique_max) {
        int64_t q = q_clique(w, deg);
        int node[kNetUnroll];
        const int c = clique_nodes(a.pin_x, lo, hi, v, node);
        if (!c) return;
        int64_t k = rp[v] + slot[p];
        if (deg <= kNetUnroll) {
#pragma unroll
            for (int u = 0; u < kNetUnroll; ++u)
                if (lo + u < hi && node[u] != v) {
                    raw[k] = raw_ent(node[u], q);
                    ++k;
                }
        } else {
            for (int b = lo; b < hi; ++b) {
                int u = a.pin_x[b];
                if (u == v) continue;
                raw[k] = raw_ent(u, q);
                ++k;
            }
        }
    } else {
        int64_t q = q_star(w, deg);
        int z = a.first_star + a.star_rank[e];
        int64_t k = rp[v] + slot[p];
        raw[k] = raw_ent(z, q);
        int64_t kz = rp[z] + (p - lo);
        raw[kz] = raw_ent(v, q);
    }
}

// Row classes by entry count: 0 (<= 1), 1 (<= 8), 2 (<= 16), 3 (<= 32),
// 4 (<= 64), 5 (<= kMidRow), 6 (longer); classes 1-4 are sorted by 8, 16, 32
// and 64 lanes per row, 5 and 6 by workgroups of kMidBT and kLongBT threads.
constexpr int kSortClasses = 7;
constexpr int kMidRow = 2048;
__device__ __forceinline__ int row_class(int64_t c) {
    return c <= 1 ? 0 : c <= 8 ? 1 : c <= 16 ? 2 : c <= 32 ? 3 : c <= 64 ? 4 : c <= kMidRow ? 5 : 6;
}

// The rows' first slots, and the rows listed by class (ascending within one).
struct RowScan {
    static constexpr int K = 4;
    static constexpr bool kTotal = true, kHeavy = false;
    using Raw = int32_t;        // the row's count and one, 0 for no row
    const int32_t* cnt;
    int32_t n;
    int64_t* rp;                // [n + 1]
    int32_t* list;              // [n]
    int32_t* start;             // [kSortClasses + 1]
    __device__ int32_t first(int64_t r) const { return cnt[r] + 1; }
    __device__ int32_t again(int64_t r) const { return first(r); }
    __device__ Pack<4> pack(int32_t c1) const {
        const int c = c1 > 0 ? c1 - 1 : 0, k = row_class(c);
        Pack<4> p{{c, 0, 0, 0}};
#pragma unroll
        for (int q = 1; q < kSortClasses; ++q)
            if (k == q) p.v[1 + (q - 1) / 2] = (q - 1) & 1 ? int64_t(1) << 32 : 1;
        return p;
    }
    // of the rows counted in t (of which there are `rows`), those of class k
    __device__ static int32_t of(const Pack<4>& t, int64_t rows, int k) {
        int64_t others = 0;
        int32_t own = 0;
#pragma unroll
        for (int q = 1; q < kSortClasses; ++q) {
            const int32_t c = (q - 1) & 1 ? pack_hi(t.v[1 + (q - 1) / 2]) : pack_lo(t.v[1 + (q - 1) / 2]);
            others += c;
            own = q == k ? c : own;
        }
        return k ? own : static_cast<int32_t>(rows - others);
    }
    __device__ void item(int64_t r, int32_t c1, const Pack<4>& before, const Pack<4>& total) const {
        rp[r] = before.v[0];
        const int k = row_class(c1 - 1);
        int32_t at = of(before, r, k);
#pragma unroll
        for (int q = 0; q < kSortClasses - 1; ++q) at += q < k ? of(total, n, q) : 0;
        list[at] = static_cast<int32_t>(r);
    }
    __device__ void done(const Pack<4>& total) const {
        rp[n] = total.v[0];
        int32_t at = 0;
        for (int q = 0; q <= kSortClasses; ++q) {
            start[q] = at;
            if (q < kSortClasses) at += of(total, n, q);
        }
    }
};

// The sorted rows' arrays: row r's raw entries are raw[rp[r]..+cnt[r]); its
// merged entries go to the same slots of scol and sq, their number to len and
// their weight sum to qdeg.
struct SortArgs {
    const int32_t* cnt;
    const int64_t* rp;
    const RawEnt* raw;
    int32_t* scol;
    int64_t* sq;
    int32_t* len;
    int64_t* qdeg;
};

__device__ __forceinline__ void row_done(const SortArgs& a, int r, int len, int64_t q) {
    a.len[r] = len;
    a.qdeg[r] = q;
}

// Rows with at most one entry: copy through.
__device__ __forceinline__ void sort_trivial(const SortArgs& a, const int32_t* rows, int32_t nrows, int32_t block) {
    const int64_t i = static_cast<int64_t>(block) * kBT + threadIdx.x;
    if (i >= nrows) return;
    const int r = rows[i], c = a.cnt[r];
    int64_t q = 0;
    if (c == 1) {
        const int64_t base = a.rp[r];
        const RawEnt e = a.raw[base];
        a.scol[base] = e.col;
        a.sq[base] = e.q;
        q = e.q;
    }
    row_done(a, r, c, q);
}

// The lanes that keep the smaller key in step (K, J) of the bitonic network
// over groups of G lanes.
template <int G>
constexpr uint64_t bitonic_low(int K, int J) {
    uint64_t m = 0;
    for (int i = 0; i < kWave; ++i) {
        const int l = i & (G - 1);
        if (((l & J) == 0) == ((l & K) == 0)) m |= 1ull << i;
    }
    return m;
}

template <int G, int K, int J>
__device__ __forceinline__ int bitonic_steps(int x) {
    int a, b;
    lane_pair<J>(x, a, b);
    constexpr uint64_t low = bitonic_low<G>(K, J);
    x = __builtin_amdgcn_inverse_ballot_w64(low) ? (a < b ? a : b) : (a < b ? b : a);
    if constexpr (J > 1) return bitonic_steps<G, K, J / 2>(x);
    else if constexpr (K < G) return bitonic_steps<G, 2 * K, K>(x);
    else return x;
}

// G lanes per row (G = 8, 16, 32 or 64): bitonic sort by column across the
// lanes, then equal columns merged by exact integer sums.  Narrow: the column
// ids leave room for a lane index beside them in 31 bits.
// What bounds it: the vector instructions of a wave (a row of few entries
// takes the whole of its lanes through the network) beside 28 bytes of memory
// an entry, so the exchanges are part of the comparisons (no shuffles), the
// network's directions are constants, and the run sums take as many steps as
// the wave's longest run of equal columns needs.
// 108 us at 600k cells (gift), against 135 with shuffles and full-length sums;
// 32 for 44 at 210k, 12.6 for 17.8 at 73k, 415 for 445 at 2.2M.
template <int G, bool Narrow>
__device__ __forceinline__ void sort_group(const SortArgs& a, const int32_t* rows, int32_t nrows, int32_t block) {
    int64_t gid = (static_cast<int64_t>(block) * kBT + threadIdx.x) / G;
    int l = threadIdx.x & (G - 1);
    int lane = lane_id();
    int gbase = lane - l;      // first lane of this group inside the wave
    bool valid_row = gid < nrows;
    int r = valid_row ? rows[gid] : 0;
    int len = valid_row ? a.cnt[r] : 0;
    int64_t base = valid_row ? a.rp[r] : 0;
    int key = 0x7fffffff;
    int64_t q = 0;
    if (l < len) {
        const RawEnt e = a.raw[base + l];
        key = e.col;
        q = e.q;
    }
    if constexpr (Narrow) {
        // one 32-bit key per lane, (column, lane) packed: unique, so the
        // network moves the key alone and each lane then fetches the weight
        // of the entry it ended up with
        constexpr int LB = G == 8 ? 3 : G == 16 ? 4 : G == 32 ? 5 : 6;
        const int ck = bitonic_steps<G, 2, 1>(l < len ? ((key << LB) | l) : 0x7fffffff);
        q = __shfl(q, gbase + (ck & (G - 1)));
        key = l < len ? (ck >> LB) : 0x7fffffff;
    } else {
#pragma unroll
        for (int k = 2; k <= G; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                int pk = __shfl_xor(key, j);
                int64_t pq = __shfl_xor(q, j);
                bool up = (l & k) == 0;
                bool lower = (l & j) == 0;
                bool take = lower ? (up ? (pk < key) : (pk > key)) : (up ? (pk > key) : (pk < key));
                if (take) {
                    key = pk;
                    q = pq;
                }
            }
        }
    }
    const bool live = l < len;
    if (!live) q = 0;
    const int prev = dpp<kDppPrev>(key), next = dpp<kDppNext>(key);
    const bool head = live && (l == 0 || prev != key);
    const bool tail = live && (l + 1 == len || next != key);
    // the row's weight sum
    int64_t total = q;
    total = pair_sum<1>(total);
    total = pair_sum<2>(total);
    total = pair_sum<4>(total);
    if constexpr (G > 8) total = pair_sum<8>(total);
    if constexpr (G > 16) total = pair_sum<16>(total);
    if constexpr (G > 32) total = pair_sum<32>(total);
    // sums of the runs of equal columns, complete at their last lanes; done
    // with the first distance that no lane has an equal column at
    int64_t sum = q;
    for (int d = 1; d < G; d <<= 1) {
        const int from = l >= d ? lane - d : lane;
        const int there = __shfl(key, from);
        const bool same = live && l >= d && there == key;
        if (!__any(same)) break;
        const int64_t add = __shfl(sum, from);
        sum += same ? add : 0;
    }
    const uint64_t hm = __ballot(head);
    // the runs that start at or before the lane, of which those of the groups below
    const int upto = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(hm >> 32),
                                               __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(hm), head ? 1 : 0));
    const int idx = upto - __popcll(hm & ((1ull << gbase) - 1ull)) - 1;
    if (tail) {
        a.scol[base + idx] = key;
        a.sq[base + idx] = sum;
    }
    if (valid_row && l == G - 1) row_done(a, r, idx + 1, total);
}

// The five classes of at most 64 entries in one launch: workgroups [b[k],
// b[k+1]) take class k, the wide ones first.
struct SortLists {
    const int32_t* rows[5];
    int32_t n[5];
    int32_t b[6];
};

template <bool Narrow>
__global__ void __launch_bounds__(kBT) k_sort_rows(SortArgs a, SortLists s) {
    const int32_t b = static_cast<int32_t>(blockIdx.x);
    if (b < s.b[1]) sort_group<64, Narrow>(a, s.rows[0], s.n[0], b);
    else if (b < s.b[2]) sort_group<32, Narrow>(a, s.rows[1], s.n[1], b - s.b[1]);
    else if (b < s.b[3]) sort_group<16, Narrow>(a, s.rows[2], s.n[2], b - s.b[2]);
    else if (b < s.b[4]) sort_group<8, Narrow>(a, s.rows[3], s.n[3], b - s.b[3]);
    else sort_trivial(a, s.rows[4], s.n[4], b - s.b[4]);
}

// One workgroup per longer row: sort of (column, slot) keys -- in LDS when
// the row fits `lds_keys` (dynamic shared memory), otherwise a bitonic network
// in the row's own segment of `tkey` (global memory), with positions past the
// row end acting as +infinity -- then an ordered merge of equal columns.
// Rows reach 10^4 entries, but most have a few hundred: with kLongBT threads
// and the LDS of the longest row for each, one row a CU, the 1,700 of a
// 600k-cell netlist took 441 us.  Up to kMidRow entries they take kMidBT
// threads and 16 KB, eight rows a CU.  What bounds a row is its chain of LDS
// steps and barriers, so its tail is one pass of block scans (merge_row): 45
// us for the rows up to kMidRow and 82 for the longer ones, against 83 and 133
// with a merge that ranked BT entries at a time and added each column's
// weights one load after another (210k cells: 32 us for 60; 73k: 20 for 37).
constexpr int kLongBT = 1024;
constexpr int kMidBT = 256;

// Merge sort of a long row's keys (unique 64-bit) by one workgroup, for rows
// of at most BT * RunMax keys: thread t sorts the E keys from t E on
// in registers (odd-even transposition, fixed indices), then log2(BT)
// merge rounds double the sorted runs.  In a round each thread finds where
// its E outputs start on the merge path of its pair of runs (binary
// search), merges them into registers, and after a barrier writes them back
// in place (the thread's keys stay in v as well).  Slots past n hold ~0 and sort last.  O(n log n) LDS traffic,
// against O(n log^2 n) for the bitonic network used for longer rows.
template <int BT, int kRunMax>
__device__ __forceinline__ void block_merge_sort(const RawEnt* __restrict__ raw, int64_t base, int n, int E,
                                                 uint64_t* key, uint64_t (&v)[kRunMax]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int u = 0; u < kRunMax; ++u) {
        const int k = t + u * BT;
        const bool ok = u < E && k < n;
        const int32_t c = raw[base + (ok ? k : 0)].col;          // every load in flight at once
        v[u] = ok ? (static_cast<uint64_t>(static_cast<uint32_t>(c)) << 32) | static_cast<uint32_t>(k) : ~0ull;
    }
#pragma unroll
    for (int rnd = 0; rnd < kRunMax; ++rnd) {
#pragma unroll
        for (int u = rnd & 1; u + 1 < kRunMax; u += 2) {
            const uint64_t x = v[u], y = v[u + 1];
            v[u] = y < x ? y : x;
            v[u + 1] = y < x ? x : y;
        }
    }
#pragma unroll
    for (int u = 0; u < kRunMax; ++u)
        if (u < E) key[t * E + u] = v[u];
    __syncthreads();
    const int total = BT * E;
    for (int w = E; w < total; w <<= 1) {
        const int d0 = t * E;
        const int s = d0 / (2 * w) * (2 * w);
        const uint64_t* A = key + s;
        const uint64_t* B = key + s + w;
        const int d = d0 - s;
        int lo = d > w ? d - w : 0, hi = d < w ? d : w;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (A[mid] <= B[d - mid - 1]) lo = mid + 1;
            else hi = mid;
        }
        int i = lo, j = d - lo;
#pragma unroll
        for (int u = 0; u < kRunMax; ++u) {
            if (u < E) {
                const uint64_t a = i < w ? A[i] : ~0ull, b = j < w ? B[j] : ~0ull;
                const bool ta = j >= w || (i < w && a <= b);
                v[u] = ta ? a : b;
                i += ta ? 1 : 0;
                j += ta ? 0 : 1;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kRunMax; ++u)
            if (u < E) key[t * E + u] = v[u];
        __syncthreads();
    }
}

// A row sorted that way, and its equal columns merged: each thread counts the
// columns that start among its E keys and adds their weights (every gather in
// flight), and the weight of a column is the difference of the exact prefix
// sums where it and the next one start.
template <int BT, int RunMax>
__device__ __forceinline__ void merge_row(const SortArgs& a, int r, int64_t base, int n, int E, uint64_t* key) {
    __shared__ int64_t red[BT / kWave];
    const int t = threadIdx.x;
    uint64_t v[RunMax];
    block_merge_sort<BT, RunMax>(a.raw, base, n, E, key, v);
    uint32_t col = t > 0 ? static_cast<uint32_t>(key[t * E - 1] >> 32) : 0;
    uint32_t heads = 0;
#pragma unroll
    for (int u = 0; u < RunMax; ++u) {
        const uint32_t c = static_cast<uint32_t>(v[u] >> 32);
        if (u < E && t * E + u < n && (c != col || (t == 0 && u == 0))) heads |= 1u << u;
        col = c;
    }
    asm("" : "+v"(heads));                 // one register here and below, not what is made of it
    int64_t cols, weight, sum = 0;
    const int at = static_cast<int>(block_exclusive_scan_i64<BT>(__popc(heads), red, &cols));
    int32_t* scol = a.scol + base;
#pragma unroll
    for (int u = 0; u < RunMax; ++u)
        if (heads >> u & 1) scol[at + __popc(heads & ((1u << u) - 1))] = static_cast<int32_t>(v[u] >> 32);
    static_assert(BT * RunMax <= 1 << 16, "slots of a row");
    const RawEnt* raw = a.raw + base;
    int64_t q[RunMax];
#pragma unroll
    for (int u = 0; u < RunMax; ++u) {
        const bool ok = u < E && t * E + u < n;
        q[u] = raw[ok ? static_cast<uint32_t>(v[u]) & 0xffffu : 0].q;      // (a 32-bit offset: slots stay below 2^16)
        if (!ok) q[u] = 0;
    }
#pragma unroll
    for (int u = 0; u < RunMax; ++u) sum += q[u];
    sum = block_exclusive_scan_i64<BT>(sum, red, &weight);
    asm("" : "+v"(heads));
    // (every key has been read: the scans' barriers lie between)
    int64_t* first = reinterpret_cast<int64_t*>(key);
#pragma unroll
    for (int u = 0; u < RunMax; ++u) {
        if (heads >> u & 1) first[at + __popc(heads & ((1u << u) - 1))] = sum;
        sum += q[u];
    }
    __syncthreads();
    for (int k = t; k < cols; k += BT) a.sq[base + k] = (k + 1 < cols ? first[k + 1] : weight) - first[k];
    if (t == 0) row_done(a, r, static_cast<int>(cols), weight);
}

template <int BT, int RunMax>
__global__ void __launch_bounds__(BT) k_sort_long(SortArgs a, const int32_t* __restrict__ rows,
                                                  uint64_t* __restrict__ tkey, int lds_keys) {
    extern __shared__ uint64_t lkey[];
    __shared__ int red[BT / kWave];
    __shared__ int carry;
    __shared__ unsigned long long qtot;      // the row's weight sum (exact: integer adds)
    const RawEnt* raw = a.raw;
    int r = rows[blockIdx.x];
    int n = a.cnt[r];
    int64_t base = a.rp[r];
    // an odd number of keys a thread, where it fits, keeps the threads' runs
    // off one another's LDS banks
    int E = (n + BT - 1) / BT;
    E = (E | 1) <= RunMax && BT * (E | 1) <= lds_keys ? E | 1 : E;
    if (E <= RunMax && BT * E <= lds_keys) {                       // block-uniform
        merge_row<BT, RunMax>(a, r, base, n, E, lkey);
        return;
    }
    int P = 1;
    while (P < n) P <<= 1;
    uint64_t* key = P <= lds_keys ? lkey : tkey + base;
    for (int k = threadIdx.x; k < n; k += BT)
        key[k] = (static_cast<uint64_t>(static_cast<uint32_t>(raw[base + k].col)) << 32) | static_cast<uint32_t>(k);
    __threadfence_block();
    __syncthreads();
    for (int size = 2; size <= P; size <<= 1) {
        int half = size >> 1;
        // first comparator layer of a merge: mirror pairs
        for (int i = threadIdx.x; i < P / 2; i += BT) {
            int blk = i / half, off = i % half;
            int a = blk * size + off;
            int b = blk * size + size - 1 - off;
            if (b < n) {
                uint64_t x = key[a], y = key[b];
                if (y < x) { key[a] = y; key[b] = x; }
            }
        }
        __threadfence_block();
        __syncthreads();
        for (int h = half >> 1; h > 0; h >>= 1) {
            for (int i = threadIdx.x; i < P / 2; i += BT) {
                int a = (i / h) * 2 * h + (i % h);
                int b = a + h;
                if (b < n) {
                    uint64_t x = key[a], y = key[b];
                    if (y < x) { key[a] = y; key[b] = x; }
                }
            }
            __threadfence_block();
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) {
        carry = 0;
        qtot = 0;
    }
    __syncthreads();
    for (int t0 = 0; t0 < n; t0 += BT) {
        int k = t0 + threadIdx.x;
        uint32_t col = 0;
        bool head = false;
        if (k < n) {
            col = static_cast<uint32_t>(key[k] >> 32);
            head = (k == 0) || (static_cast<uint32_t>(key[k - 1] >> 32) != col);
        }
        int tot;
        int idx = block_rank<BT>(head, red, &tot);
        if (head) {
            int64_t s = 0;
            for (int m = k; m < n && static_cast<uint32_t>(key[m] >> 32) == col; ++m)
                s += raw[base + static_cast<uint32_t>(key[m] & 0xffffffffu)].q;
            a.scol[base + carry + idx] = static_cast<int32_t>(col);
            a.sq[base + carry + idx] = s;
            atomicAdd(&qtot, static_cast<unsigned long long>(s));
        }
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) row_done(a, r, carry, static_cast<int64_t>(qtot));
}

// Keys of a long row that one workgroup sorts in LDS: the largest power of
// two whose keys fit the per-workgroup shared memory with 1 KiB to spare.
int sort_lds_keys(int device) {
    static int cached[64] = {0};
    if (device >= 0 && device < 64 && cached[device]) return cached[device];
    hipDeviceProp_t prop;
    AHR_HIP(hipGetDeviceProperties(&prop, device));
    size_t avail = prop.sharedMemPerBlock > 1024 ? prop.sharedMemPerBlock - 1024 : 0;
    int k = 1;
    while (static_cast<size_t>(k) * 2 * sizeof(uint64_t) <= avail && k < (1 << 16)) k <<= 1;
    if (device >= 0 && device < 64) cached[device] = k;
    return k;
}

}  // namespace

void build_netlist(Graph& g, hipStream_t s) {
    ProfScope ps(kStageBuild, s);
    const ahr_netlist& nl = g.nl;
    const int32_t n_pins = nl.n_pins, n_nets = nl.n_nets, n_inst = nl.n_inst;
    const ahr_hint_params& hp = g.hp;

    // validate the device arrays
    g.counter.ensure(8, s);
    fill_i32(g.counter.p, 8, 0, s);
    int64_t nv = (n_pins > n_nets + 1) ? n_pins : static_cast<int64_t>(n_nets) + 1;
    hipLaunchKernelGGL(k_validate, dim3(grid_for(nv, kBT)), dim3(kBT), 0, s, nl.net_ptr, n_nets, nl.pin_node, n_pins,
                       n_inst, g.counter.p);
    AHR_LAUNCHED("k_validate");
    // The verdict is read together with the counts below: the kernels in
    // between index only with clamped pin nodes, so an invalid netlist reads
    // nothing out of bounds before it is rejected.

    // ranks of macro pins, star nets, big nets, macros; one read of their counts
    DevBuf<uint8_t> is_mp;
    DevBuf<int32_t> mp_rank, star_rank, big_rank, mac_rank, bs_rank;
    is_mp.ensure(static_cast<size_t>(n_pins) + 1, s);
    mp_rank.ensure(static_cast<size_t>(n_pins) + 1, s);
    star_rank.ensure(static_cast<size_t>(n_nets) + 1, s);
    big_rank.ensure(static_cast<size_t>(n_nets) + 1, s);
    bs_rank.ensure(static_cast<size_t>(n_nets) + 1, s);
    mac_rank.ensure(static_cast<size_t>(n_inst) + 1, s);
    int32_t* c = g.counter.p;      // [0] verdict, [1] macro pins, [2..4] nets, [5..6] macros
    run_scans(scan_job(PinScan{nl.pin_node, nl.node_flags, n_pins, n_inst, (hp.flags & AHR_EXPAND_MACRO_PINS) ? 1 : 0,
                               is_mp.p, mp_rank.p, c + 1},
                       n_pins),
              g.scan_tmp, s,
              scan_job(NetScan{nl.net_ptr, n_nets, hp.clique_max, star_rank.p, big_rank.p, bs_rank.p, c + 2}, n_nets),
              scan_job(MacroScan{nl.node_flags, n_inst, mac_rank.p, c + 5}, n_inst));
    int32_t cnt7[7];
    read_scalars({c, c + 1, c + 2, c + 3, c + 4, c + 5, c + 6}, cnt7, s);
    if (const int32_t bad = cnt7[0]) {
        static const char* why[] = {"", "pin_node out of [0, n_inst)", "net_ptr[0] != 0",
                                    "net_ptr[n_nets] != n_pins", "net_ptr decreasing"};
        throw Error{AHR_EINVAL, std::string("invalid netlist: ") + why[bad]};
    }
    is_mp.release(s);
    g.n_mpin = cnt7[1];
    g.n_star = cnt7[2];
    const int32_t n_big_nets = cnt7[3];
    g.n_big_stars = cnt7[4];
    g.n_macro = cnt7[5];
    g.n_movable_macro = cnt7[6];
    if ((hp.flags & AHR_MACRO_HINTS) && g.n_macro > 16384)
        throw Error{AHR_EUNSUPPORTED, "macro hints support at most 16384 macros"};

    // node ranges
    int64_t first_mpin = n_inst;
    int64_t first_star = first_mpin + g.n_mpin;
    int64_t first_mvirt = first_star + g.n_star;
    int64_t n_mv = (hp.flags & AHR_MACRO_HINTS) ? g.n_macro : 0;
    int64_t first_bvirt = first_mvirt + n_mv;
    int64_t n_bins = (hp.flags & AHR_BIN_HINTS) ? static_cast<int64_t>(hp.nbx) * hp.nby : 0;
    int64_t n_tot = first_bvirt + n_bins;
    if (n_tot >= INT32_MAX) throw Error{AHR_EUNSUPPORTED, "graph has 2^31 or more nodes"};
    g.first_mpin = static_cast<int32_t>(first_mpin);
    g.first_star = static_cast<int32_t>(first_star);
    g.first_mvirt = static_cast<int32_t>(first_mvirt);
    g.first_bvirt = static_cast<int32_t>(first_bvirt);
    g.n_bins = static_cast<int32_t>(n_bins);
    g.n_tot = static_cast<int32_t>(n_tot);
    g.n_inst = n_inst;
    const int32_t N = g.n_tot;

    // the lists, the net of every pin, then entry counts per row (parallel
    // edges counted)
    DevBuf<int32_t> pin_net, cnt, slot, big_nets;
    pin_net.ensure(static_cast<size_t>(n_pins) + 1, s);
    cnt.ensure(static_cast<size_t>(N) + 1, s);
    slot.ensure(static_cast<size_t>(n_pins) + 1, s);
    g.star_net.ensure(static_cast<size_t>(g.n_star) + 1, s);
    big_nets.ensure(static_cast<size_t>(n_big_nets) + 1, s);
    g.big_stars.ensure(static_cast<size_t>(g.n_big_stars) + 1, s);
    g.macro_ids.ensure(static_cast<size_t>(g.n_macro) + 1, s);
    g.pin_node_x.ensure(static_cast<size_t>(n_pins) + 1, s);
    g.mpin_owner.ensure(static_cast<size_t>(g.n_mpin) + 1, s);
    g.mpin_pin.ensure(static_cast<size_t>(g.n_mpin) + 1, s);
    const ListArgs la{nl.net_ptr,     nl.pin_node,    n_pins,       n_nets,         n_inst,
                      mp_rank.p,      star_rank.p,    big_rank.p,   bs_rank.p,      mac_rank.p,
                      g.pin_node_x.p, g.mpin_owner.p, g.mpin_pin.p, g.star_net.p,   big_nets.p,
                      g.big_stars.p,  g.macro_ids.p,  pin_net.p,    cnt.p,          N + 1};
    const int64_t nlist = std::max<int64_t>(std::max<int64_t>(n_pins, n_nets), static_cast<int64_t>(N) + 1);
    hipLaunchKernelGGL(k_build_lists, dim3(grid_for(nlist, kBT)), dim3(kBT), 0, s, la);
    AHR_LAUNCHED("k_build_lists");
    mp_rank.release(s);
    big_rank.release(s);
    bs_rank.release(s);
    mac_rank.release(s);
    if (n_big_nets) {
        hipLaunchKernelGGL(k_pin_net_big, dim3(n_big_nets), dim3(kBT), 0, s, big_nets.p, nl.net_ptr, pin_net.p);
        AHR_LAUNCHED("k_pin_net_big");
    }
    big_nets.release(s);
    NetArgs a{nl.net_ptr, pin_net.p, g.pin_node_x.p, nl.net_w, star_rank.p, n_nets, n_pins, hp.clique_max,
              g.first_star};
    if (n_pins)
        hipLaunchKernelGGL(k_row_counts, dim3(grid_for(n_pins, kBT)), dim3(kBT), 0, s, a, cnt.p, slot.p);
    AHR_LAUNCHED("k_row_counts");
    // the rows stay where the raw entries put them: net_off[r] is row r's
    // first slot, net_len[r] its merged entry count (set by the sorts)
    DevBuf<int64_t>& rp = g.net_off;
    rp.ensure(static_cast<size_t>(N) + 1, s);
    // (rows grouped by length class, ascending within a class)
    constexpr int K = kSortClasses;
    DevBuf<int32_t> lists, cstart;
    lists.ensure(static_cast<size_t>(N) + 1, s);
    cstart.ensure(K + 1, s);
    run_scans(scan_job(RowScan{cnt.p, N, rp.p, lists.p, cstart.p}, N), g.scan_tmp, s);
    int64_t w[K + 1];
    read_words({{rp.p + N, 1}, {cstart.p + 1, 0}, {cstart.p + 2, 0}, {cstart.p + 3, 0}, {cstart.p + 4, 0},
                {cstart.p + 5, 0}, {cstart.p + 6, 0}, {cstart.p + 7, 0}},
               w, s);
    static_assert(K == 7, "class starts read above (the first is 0)");
    const int64_t nnz_dup = w[0];
    if (nnz_dup >= INT32_MAX) throw Error{AHR_EUNSUPPORTED, "netlist expands to 2^31 or more graph entries"};
    int32_t ncls[K];
    const int32_t* cls[K];
    for (int k = 0; k < K; ++k) {
        const int64_t first = k ? w[k] : 0;
        ncls[k] = static_cast<int32_t>(w[1 + k] - first);
        cls[k] = lists.p + first;
    }

    DevBuf<int32_t>& scol = g.net_col;
    DevBuf<int32_t>& ucnt = g.net_len;
    DevBuf<RawEnt> raw;
    DevBuf<int64_t>& sq = g.net_q;
    raw.ensure(static_cast<size_t>(nnz_dup) + 1, s);
    if (n_pins)
        hipLaunchKernelGGL(k_scatter, dim3(grid_for(n_pins, kBT)), dim3(kBT), 0, s, a, rp.p, slot.p, raw.p);
    AHR_LAUNCHED("k_scatter");
    slot.release(s);
    pin_net.release(s);
    star_rank.release(s);

    // per-row sort + merge by length class
    scol.ensure(static_cast<size_t>(nnz_dup) + 1, s);
    sq.ensure(static_cast<size_t>(nnz_dup) + 1, s);
    ucnt.ensure(static_cast<size_t>(N) + 1, s);
    g.qdeg.ensure(static_cast<size_t>(N) + 1, s);
    const SortArgs sa{cnt.p, rp.p, raw.p, scol.p, sq.p, ucnt.p, g.qdeg.p};
    // rows of up to 64 entries sort (column, lane) pairs packed in 32 bits
    const bool narrow = N < (1 << 25);
    SortLists sl{};
    const int lanes[5] = {64, 32, 16, 8, 1};
    for (int k = 0; k < 5; ++k) {
        sl.rows[k] = cls[4 - k];
        sl.n[k] = ncls[4 - k];
        const int64_t t = static_cast<int64_t>(ncls[4 - k]) * lanes[k];
        sl.b[k + 1] = sl.b[k] + static_cast<int32_t>((t + kBT - 1) / kBT);
    }
    if (sl.b[5]) {
        hipLaunchKernelGGL((narrow ? k_sort_rows<true> : k_sort_rows<false>), dim3(sl.b[5]), dim3(kBT), 0, s, sa, sl);
        AHR_LAUNCHED("k_sort_rows");
    }
    if (ncls[5]) {
        hipLaunchKernelGGL((k_sort_long<kMidBT, kMidRow / kMidBT>), dim3(ncls[5]), dim3(kMidBT),
                           kMidRow * sizeof(uint64_t), s, sa, cls[5], static_cast<uint64_t*>(nullptr), kMidRow);
        AHR_LAUNCHED("k_sort_long mid");
    }
    if (ncls[6]) {
        DevBuf<uint64_t> tkey;
        tkey.ensure(static_cast<size_t>(nnz_dup) + 1, s);
        const int lds_keys = sort_lds_keys(g.device);
        hipLaunchKernelGGL((k_sort_long<kLongBT, 16>), dim3(ncls[6]), dim3(kLongBT),
                           static_cast<size_t>(lds_keys) * sizeof(uint64_t), s, sa, cls[6], tkey.p, lds_keys);
        AHR_LAUNCHED("k_sort_long");
        tkey.release(s);
    }
    raw.release(s);
    // the rows the execution-order copy gives a workgroup each (it takes
    // those still above kShortRow entries)
    g.n_long_nodes = ncls[5] + ncls[6];
    g.long_nodes.ensure(static_cast<size_t>(g.n_long_nodes) + 1, s);
    if (g.n_long_nodes)
        AHR_HIP(hipMemcpyAsync(g.long_nodes.p, cls[5], static_cast<size_t>(g.n_long_nodes) * sizeof(int32_t),
                               hipMemcpyDeviceToDevice, s));

    // The merged rows stay in place (no compaction): slots past a row's
    // merged count are unused.  The arrays hold the raw count; the exact
    // entry count is read later with other sizes.
    g.nnz_net = -1;
    g.nnz_cap = static_cast<int32_t>(nnz_dup);
    lists.release(s);
    cstart.release(s);
    cnt.release(s);
}

}  // namespace ahr
