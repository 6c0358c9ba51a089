// Execution layout of the filter.  Instance ids arrive in netlist order,
// which carries no locality, so neighbour gathers of the SpMM hop would each
// touch a different cache line.  The filter therefore streams rows in an
// execution order: instances sorted by a stable sort on the Hilbert-curve
// index of their position on a 1024 x 1024 grid over the die, columns
// renumbered to match.  The macro pin nodes and the star nodes stay in their
// own id ranges but are ordered the same way inside them (a macro pin by its
// pin position, a star by the position of its net's first pin), so that the
// rows gathering a run of them, and their own rows, touch few cache lines;
// the virtual nodes keep their canonical ids.  Consecutive rows are then spatial neighbours, so the
// rows of one workgroup gather from few, shared cache lines, and every
// aligned power-of-two block of the grid (a bin of a 2^k x 2^k bin grid) is
// one contiguous range of rows.  Inside each aligned window of 64 rows (the
// rows of one workgroup of the hop) the rows are then ordered by netlist
// row length, so the rows that share a wave need about the same number of
// entry batches and the window stays one spatial neighbourhood.  The
// netlist rows are copied into that order, the entries of each short row
// sorted by their renumbered column (so a row's gathers also walk the
// layout in order; the summation order is fixed by the inputs and the first
// placement); the hint rows are built in it directly.  The canonical netlist
// CSR stays for export; the order is set once per graph from the first
// placement seen.
//
// A placement whose positions say little about the netlist (uniformly
// drawn ones, or a low-order smoothing of them) gives a Hilbert order with
// no locality.  On request (AHR_LAYOUT_NETLIST) the instances take a
// netlist order instead: Cuthill-McKee levels over the instance-to-instance
// netlist edges (star and macro pin nodes left out, since a big net reaches
// across the die), a node's rank following its lowest-ranked parent,
// siblings in id order; macro pin and star rows follow the lowest rank among
// their instance neighbours.  With AHR_LAYOUT_AUTO the Hilbert order is kept
// when at least a quarter of a sample of its instance-to-instance entries lie
// within n_inst/64 rows (at least 256) of their row (a random order puts
// about 1/32 of them there), else the netlist order is taken.
#include "ahr_internal.hpp"
#include "device_util.hpp"
#include "scan.hpp"

namespace ahr {

namespace {

constexpr int kBT = 256;
constexpr int kGridBits = 10;    // 1024 x 1024 layout grid -> 20-bit Hilbert keys
constexpr int kKeyBits = 22;     // the node range (instance, macro pin, star) above them
constexpr int kDigitBits = 11;   // sorted as two stable 11-bit digit passes

// Hilbert-curve index of grid cell (x, y) on the 2^kGridBits square grid:
// at each level the quadrant's position along the curve, then the cell's
// coordinates reflected into that quadrant's orientation.
__device__ __forceinline__ int hilbert_index(int x, int y) {
    int d = 0;
    for (int s = 1 << (kGridBits - 1); s > 0; s >>= 1) {
        const int rx = (x & s) ? 1 : 0, ry = (y & s) ? 1 : 0;
        d += s * s * ((3 * rx) ^ ry);
        if (ry == 0) {
            if (rx == 1) {
                x = s - 1 - x;
                y = s - 1 - y;
            }
            const int t = x;
            x = y;
            y = t;
        }
    }
    return d;
}

struct KeyArgs {
    const float* pos;            // instance positions, ncols per row
    int ncols;
    int32_t n_inst, first_star, first_mvirt;
    const int32_t* mpin_pin;     // pin of each macro pin node
    const int32_t* star_net;     // net of each star node
    const int32_t* net_ptr;
    const int32_t* pin_node;     // instance of each pin
    const int32_t* pin_node_x;   // node of each pin (macro pins expanded)
    const float* pin_off;
    float xl, yl, sx, sy;
};

// Position of pin p: its instance's, plus the pin offset where the pin is
// its own node.
__device__ __forceinline__ float2 pin_pos(const KeyArgs& a, int p) {
    const int v = a.pin_node[p];
    float x = a.pos[static_cast<int64_t>(v) * a.ncols], y = a.pos[static_cast<int64_t>(v) * a.ncols + 1];
    if (a.pin_node_x[p] >= a.n_inst) {
        x += a.pin_off[2 * p];
        y += a.pin_off[2 * p + 1];
    }
    return make_float2(x, y);
}

// Sort key of node i < first_mvirt: its range above the Hilbert index of
// its position.
__global__ void k_layout_keys(KeyArgs a, int32_t* __restrict__ key) {
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= a.first_mvirt) return;
    float2 q;
    int range;
    if (i < a.n_inst) {
        q = make_float2(a.pos[i * a.ncols], a.pos[i * a.ncols + 1]);
        range = 0;
    } else if (i < a.first_star) {
        q = pin_pos(a, a.mpin_pin[i - a.n_inst]);
        range = 1;
    } else {
        q = pin_pos(a, a.net_ptr[a.star_net[i - a.first_star]]);
        range = 2;
    }
    const int m = (1 << kGridBits) - 1;
    float fx = floorf((q.x - a.xl) * a.sx);
    float fy = floorf((q.y - a.yl) * a.sy);
    int gx = !(fx > 0.f) ? 0 : (fx >= static_cast<float>(m) ? m : static_cast<int>(fx));
    int gy = !(fy > 0.f) ? 0 : (fy >= static_cast<float>(m) ? m : static_cast<int>(fy));
    key[i] = (range << (2 * kGridBits)) | hilbert_index(gx, gy);
}

// perm and iperm from the sorted order `in`.  The instances take a stable
// sort of each aligned window of kLenWindow positions by netlist row length
// (one wave per window): the rank of an element is the number of elements of
// its window with a smaller length, or the same length and an earlier
// position.  The macro pins and stars stay as sorted; the virtual rows (from
// n_perm on) map to themselves.
constexpr int kLenWindow = 64;

__global__ void __launch_bounds__(kLenWindow) k_window_sort(int32_t n_inst, int32_t n_perm, int32_t n_tot,
                                                            const int32_t* __restrict__ in,
                                                            const int32_t* __restrict__ net_len,
                                                            int32_t* __restrict__ perm, int32_t* __restrict__ iperm) {
    __shared__ int32_t wlen[kLenWindow];
    const int t = threadIdx.x;
    const int32_t windows = (n_inst + kLenWindow - 1) / kLenWindow;
    if (static_cast<int32_t>(blockIdx.x) >= windows) {
        const int64_t r = n_inst + static_cast<int64_t>(blockIdx.x - windows) * kLenWindow + t;
        if (r >= n_tot) return;
        const int32_t v = r < n_perm ? in[r] : static_cast<int32_t>(r);
        perm[r] = v;
        iperm[v] = static_cast<int32_t>(r);
        return;
    }
    const int32_t j = static_cast<int32_t>(blockIdx.x) * kLenWindow + t;
    int32_t id = 0, len = INT32_MAX;                 // positions past n_inst sort last and are not written
    if (j < n_inst) {
        id = in[j];
        len = net_len[id];
    }
    wlen[t] = len;
    __syncthreads();
    int rank = 0;
    for (int u = 0; u < kLenWindow; ++u) {
        const int32_t o = wlen[u];
        rank += (o < len || (o == len && u < t)) ? 1 : 0;
    }
    if (j < n_inst) {
        const int32_t r = static_cast<int32_t>(blockIdx.x) * kLenWindow + rank;
        perm[r] = id;
        iperm[id] = r;
    }
}

// Per execution row, from its node: the netlist row length, scanned into the
// row offsets, the row weight sum, for the macro pin and star rows what the
// expansion reads (a macro pin's owner instance and pin offset, a star's
// net), and for the instances what every hint round reads in row order (area
// and class, baseWeight).
struct ExecRowScan {
    static constexpr int K = 1;
    static constexpr bool kTotal = false, kHeavy = true;
    using Raw = Pack<1>;
    __device__ Pack<1> pack(const Pack<1>& p) const { return p; }
    int32_t n_tot, n_inst, first_star, first_mvirt;
    const int32_t* perm;
    const int32_t* net_len;
    const int64_t* qdeg;
    const int32_t* mpin_pin;
    const int32_t* pin_node;
    const float* pin_off;
    const int32_t* star_net;
    const uint8_t* flags;
    const float* size;
    int64_t* xqdeg;
    int4* xmpin;
    int32_t* xstar_net;
    int64_t* xcell;             // or null: no hints will be built
    double* xbase_w;
    int32_t* rp;                // [n_tot + 1]; the lengths until the rows are placed
    __device__ Pack<1> first(int64_t r) const {
        const int v = perm[r], l = net_len[v];
        const int64_t q = qdeg[v];
        rp[r] = l;
        xqdeg[r] = q;
        if (r < n_inst) {
            if (!xcell) return {{l}};
            int64_t c = kCellOther;
            if ((flags[v] & (AHR_NODE_FIXED | AHR_NODE_MACRO)) == 0) {
                const double area = static_cast<double>(size[2 * v]) * static_cast<double>(size[2 * v + 1]);
                c = static_cast<int64_t>(__builtin_rint(area * kAreaQ)) * 4 + (q > 0 ? kCellHint : kCellStd);
            }
            xcell[r] = c;
            // Section V: baseWeight, the mean weight of the instance's netlist entries
            xbase_w[r] = l > 0 && q != 0 ? (static_cast<double>(q) * 0x1p-32) / static_cast<double>(l) : 0.0;
        } else if (r < first_star) {
            const int p = mpin_pin[v - n_inst];
            xmpin[r - n_inst] =
                make_int4(pin_node[p], __float_as_int(pin_off[2 * p]), __float_as_int(pin_off[2 * p + 1]), 0);
        } else if (r < first_mvirt) {
            xstar_net[r - first_star] = star_net[v - first_star];
        }
        return {{l}};
    }
    __device__ Pack<1> again(int64_t r) const { return {{rp[r]}}; }
    __device__ void item(int64_t r, const Pack<1>&, const Pack<1>& before, const Pack<1>&) const {
        rp[r] = static_cast<int32_t>(before.v[0]);
    }
    __device__ void done(const Pack<1>& total) const { rp[n_tot] = static_cast<int32_t>(total.v[0]); }
};

// Execution-order netlist rows: each row copies its canonical row's
// entries with columns renumbered and weights as float32.  Rows of at most
// kShortRow entries are put in ascending order of the renumbered column, so
// that the lanes of a row gather neighbouring nodes in turn (a row's columns
// are distinct, so an entry's place is the count of smaller ones).  Longer
// rows keep their canonical entry order and have one workgroup each
// (k_exec_net_long).
constexpr int kShortRow = 64;

__device__ __forceinline__ int2 exec_entry(int32_t c, int64_t q, const int32_t* iperm) {
    return make_int2(iperm[c], f_bits(static_cast<float>(static_cast<double>(q) * 0x1p-32)));
}

// kExecRows consecutive rows a workgroup, one lane an entry: their short rows'
// entries are numbered through, so that no lane idles on a short row (with 8
// lanes a row and 8 slots a lane, which covers the longest row, six of seven
// loads were repeats).  What bounds it are the lines it fetches, 2.1 GB at 2.2M
// cells: parts of 128-byte lines at each canonical row's ends and at each
// renumbered column; neighbouring rows share columns, so each XCD takes a
// contiguous range of them.  569 -> 406 us at 2.2M cells (456 with the rows
// dealt over the XCDs), 149 -> 122 at 600k, 48 -> 35 at 210k, 24 -> 20 at 73k.
constexpr int kExecRows = 64;
constexpr int kExecUnroll = 4;

__global__ void __launch_bounds__(kBT) k_exec_net(int32_t n_tot, const int32_t* __restrict__ perm,
                                                  const int32_t* __restrict__ iperm, const int64_t* __restrict__ off,
                                                  const int32_t* __restrict__ col, const int64_t* __restrict__ q,
                                                  const int32_t* __restrict__ xrp, int2* __restrict__ xent) {
    constexpr int L = 4;                                        // a row's slots are a multiple of L
    static_assert(kExecRows == kWave && kShortRow % L == 0 && kBT == L * kExecRows, "layout of the slots");
    __shared__ int4 cols[kExecRows * kShortRow / L];
    __shared__ uint32_t owner[kExecRows * kShortRow / L];       // the row of L slots
    __shared__ int32_t at[kExecRows + 1], end[kExecRows];       // a row's first slot and the end of its entries
    __shared__ int32_t dst[kExecRows];
    __shared__ int64_t src[kExecRows];                          // where slot 0 would be in col and q
    const int t = threadIdx.x;
    const int64_t r0 = xcd_tile(blockIdx.x, gridDim.x) * kExecRows;
    if (t < kExecRows) {
        const int64_t r = r0 + t < n_tot ? r0 + t : n_tot - 1;
        const int d = xrp[r];
        int len = xrp[r + 1] - d;
        if (r0 + t >= n_tot || len > kShortRow) len = 0;
        const int64_t a = off[perm[r]];
        const int slots = (len + L - 1) / L * L;
        int sum = slots;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int x = __shfl_up(sum, o);
            sum += t >= o ? x : 0;
        }
        at[t] = sum - slots;
        if (t == kExecRows - 1) at[kExecRows] = sum;
        end[t] = sum - slots + len;
        dst[t] = d;
        src[t] = a - (sum - slots);
    }
    __syncthreads();
    for (int k = at[t / L] / L + t % L; k < at[t / L + 1] / L; k += L) owner[k] = t / L;
    __syncthreads();
    const int n = at[kExecRows];
    if (n == 0) return;
    constexpr int U = kExecUnroll, kPasses = kExecRows * kShortRow / (kBT * U);
    static_assert(kExecRows * kShortRow % (kBT * U) == 0, "whole passes");
    int32_t* mine = reinterpret_cast<int32_t*>(cols);
    int w[kPasses][U];
#pragma unroll
    for (int h = 0; h < kPasses; ++h) {
        const int k0 = h * kBT * U + t;
        if (h * kBT * U < n) {                                  // workgroup-uniform
            int32_t c[U];
            int64_t v[U];
            bool live[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * kBT < n ? k0 + u * kBT : n - 1;
                const int o = owner[k / L];
                live[u] = k < end[o];
                const int64_t e = src[o] + (live[u] ? k : end[o] - 1);
                c[u] = col[e];
                v[u] = q[e];
            }
            int32_t m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = iperm[c[u]];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[h][u] = f_bits(static_cast<float>(static_cast<double>(v[u]) * 0x1p-32));
                if (k0 + u * kBT < n) mine[k0 + u * kBT] = live[u] ? m[u] : INT32_MAX;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kPasses; ++h) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = h * kBT * U + t + u * kBT;
            if (k < n) {
                const int o = owner[k / L], m = mine[k];
                int rank = 0;
                for (int j = at[o] / L; j < at[o + 1] / L; ++j) {
                    const int4 y = cols[j];
                    rank += (y.x < m ? 1 : 0) + (y.y < m ? 1 : 0) + (y.z < m ? 1 : 0) + (y.w < m ? 1 : 0);
                }
                if (k < end[o]) xent[static_cast<int64_t>(dst[o]) + rank] = make_int2(m, w[h][u]);
            }
        }
    }
}

// The longer rows, one workgroup per node of the build's list (the nodes
// whose rows may be that long).
__global__ void __launch_bounds__(kBT) k_exec_net_long(const int32_t* __restrict__ nodes,
                                                       const int32_t* __restrict__ iperm,
                                                       const int64_t* __restrict__ off, const int32_t* __restrict__ col,
                                                       const int64_t* __restrict__ q, const int32_t* __restrict__ xrp,
                                                       int2* __restrict__ xent) {
    const int v = nodes[blockIdx.x], r = iperm[v];
    const int d = xrp[r], len = xrp[r + 1] - d;
    if (len <= kShortRow) return;
    const int64_t a = off[v];
    for (int k = threadIdx.x; k < len; k += kBT) xent[d + k] = exec_entry(col[a + k], q[a + k], iperm);
}


// ---------------------------------------------------------------- netlist order

constexpr int kCmGrid = 1024;       // workgroups of the level kernels (grid-stride over the level)
constexpr int kSample = 64;         // every kSample-th instance row is tested

struct CmArgs {
    int32_t n_inst;
    const int64_t* off;    // canonical netlist rows: off, merged length, columns
    const int32_t* len;
    const int32_t* col;
    unsigned long long* lk;  // [n_inst] BFS level (high word) above the rank of the
                             // lowest-ranked parent; all ones while unvisited
    int32_t* rank;         // [n_inst] position in the order, -1 unplaced
    int32_t* order;        // [n_inst] rank -> instance
    int32_t* cnt;          // [n_inst] children per rank (the current level's ranks)
    const int32_t* scn;    // exclusive scan of cnt ([n_inst] + total)
    int32_t* bnd;          // [0] lo, [1] hi: ranks of the current level; [2] start node
};

__global__ void k_cm_init(CmArgs a) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < a.n_inst) {
        a.lk[v] = ~0ull;
        a.rank[v] = -1;
        a.cnt[v] = 0;
    }
    if (v == 0) a.bnd[2] = INT32_MAX;
}

// The start: the lowest instance with an instance neighbour (one atomic per
// wave).
__global__ void __launch_bounds__(kBT) k_cm_start(CmArgs a) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    int best = INT32_MAX;
    if (v < a.n_inst) {
        const int64_t o = a.off[v];
        const int l = a.len[v];
        for (int k = 0; k < l; ++k)
            if (a.col[o + k] < a.n_inst) {
                best = static_cast<int>(v);
                break;
            }
    }
    best = wave_min(best);
    // (a wave whose candidate cannot lower the current one skips the atomic:
    // the start is nearly always among the first ids)
    if (lane_id() == 0 && best < __hip_atomic_load(&a.bnd[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMin(&a.bnd[2], best);
}

__global__ void k_cm_seed(CmArgs a) {
    int v0 = a.bnd[2];
    if (v0 == INT32_MAX) v0 = 0;            // no instance edges: the order is the id order
    a.lk[v0] = 0ull;
    a.rank[v0] = 0;
    a.order[0] = v0;
    a.bnd[0] = 0;
    a.bnd[1] = 1;
}

// The level kernels give each row of the level kCmLanes lanes, which take
// its entries in turn; the rows of a level are strided over the grid.
constexpr int kCmLanes = 8;

// The packed word of a node of level k + 1 whose lowest-ranked parent is rank i.
__device__ __forceinline__ unsigned long long cm_word(int32_t k, int64_t i) {
    return (static_cast<unsigned long long>(k + 1) << 32) | static_cast<unsigned>(i);
}

__device__ __forceinline__ bool cm_child(const CmArgs& a, int c, int32_t k, int64_t i) {
    return c < a.n_inst && a.lk[c] == cm_word(k, i);
}

// Level k (ranks [lo, hi)): every unvisited instance neighbour joins level
// k + 1 and keeps the lowest rank among its parents, both by one 64-bit
// minimum (an earlier level's word is below every level k + 1 word, an
// unvisited node's above).
__global__ void __launch_bounds__(256) k_cm_expand(CmArgs a, int32_t k) {
    const int lo = a.bnd[0], hi = a.bnd[1];
    const int ln = threadIdx.x & (kCmLanes - 1);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * (blockDim.x / kCmLanes);
    for (int64_t i = lo + (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kCmLanes; i < hi;
         i += stride) {
        const int u = a.order[i];
        const int64_t o = a.off[u];
        const int l = a.len[u];
        const unsigned long long w = cm_word(k, i);
        for (int j = ln; j < l; j += kCmLanes) {
            const int c = a.col[o + j];
            if (c < a.n_inst && a.lk[c] > w) atomicMin(&a.lk[c], w);
        }
    }
}

// Children of each rank of the level: its neighbours whose lowest parent it is.
__global__ void __launch_bounds__(256) k_cm_count(CmArgs a, int32_t k) {
    const int lo = a.bnd[0], hi = a.bnd[1];
    const int ln = threadIdx.x & (kCmLanes - 1);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * (blockDim.x / kCmLanes);
    for (int64_t i = lo + (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kCmLanes; i < hi;
         i += stride) {
        const int u = a.order[i];
        const int64_t o = a.off[u];
        const int l = a.len[u];
        int n = 0;
        for (int j = ln; j < l; j += kCmLanes) n += cm_child(a, a.col[o + j], k, i) ? 1 : 0;
#pragma unroll
        for (int m = kCmLanes / 2; m > 0; m >>= 1) n += __shfl_xor(n, m);   // the row's lanes
        if (ln == 0) a.cnt[i] = n;
    }
}

// Ranks of level k + 1: the children of rank i follow those of the ranks
// before it, each parent's in ascending id (its row is column-sorted; the
// row's lanes place each batch of kCmLanes entries by a ballot).
__global__ void __launch_bounds__(256) k_cm_assign(CmArgs a, int32_t k) {
    const int lo = a.bnd[0], hi = a.bnd[1];
    const int base0 = a.scn[lo];
    const int ln = threadIdx.x & (kCmLanes - 1);
    const int gb = lane_id() & ~(kCmLanes - 1);              // the row's first lane in the wave
    const int64_t stride = static_cast<int64_t>(gridDim.x) * (blockDim.x / kCmLanes);
    for (int64_t i = lo + (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kCmLanes; i < hi;
         i += stride) {
        const int u = a.order[i];
        const int64_t o = a.off[u];
        const int l = a.len[u];
        int r = hi + (a.scn[i] - base0);
        for (int j0 = 0; j0 < l; j0 += kCmLanes) {
            const int j = j0 + ln;
            int c = 0;
            bool f = false;
            if (j < l) {
                c = a.col[o + j];
                f = cm_child(a, c, k, i);
            }
            const unsigned gm = static_cast<unsigned>(__ballot(f) >> gb) & ((1u << kCmLanes) - 1u);
            if (f) {
                const int p = r + __popc(gm & ((1u << ln) - 1u));
                a.rank[c] = p;
                a.order[p] = c;
            }
            r += __popc(gm);
        }
    }
}

// The next level's rank range.
__global__ void k_cm_next(CmArgs a) {
    const int lo = a.bnd[0], hi = a.bnd[1];
    const int nchild = a.scn[hi] - a.scn[lo];
    a.bnd[0] = hi;
    a.bnd[1] = hi + nchild;
}

// Instances the levels never reached (other components, isolated ones):
// after the reached ones, in id order.
__global__ void k_cm_unplaced(int32_t n, const int32_t* __restrict__ rank, int32_t* __restrict__ flag) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < n) flag[v] = rank[v] < 0 ? 1 : 0;
}

__global__ void k_cm_append(int32_t n, const int32_t* __restrict__ flag, const int32_t* __restrict__ pos,
                            const int32_t* __restrict__ bnd, int32_t* __restrict__ rank) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < n && flag[v]) rank[v] = bnd[1] + pos[v];
}

// Sort keys of the netlist order (24 bits: range above the rank): an
// instance's own rank, a macro pin's or star's lowest instance-neighbour
// rank (n_inst if none; one wave per such row); low 12 bits to `lo`.
__global__ void k_cm_keys(int32_t n_inst, const int32_t* __restrict__ rank, int32_t* __restrict__ key) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < n_inst) key[v] = rank[v];
}

__global__ void __launch_bounds__(kBT) k_cm_keys_aux(int32_t n_inst, int32_t np, int32_t first_star,
                                                     const int64_t* __restrict__ off,
                                                     const int32_t* __restrict__ len,
                                                     const int32_t* __restrict__ col,
                                                     const int32_t* __restrict__ rank,
                                                     int32_t* __restrict__ key) {
    const int64_t v = n_inst + (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    if (v >= np) return;                                   // wave-uniform
    const int64_t o = off[v];
    const int l = len[v];
    int r = n_inst;
    for (int j = lane_id(); j < l; j += kWave) {
        const int c = col[o + j];
        if (c < n_inst) r = rank[c] < r ? rank[c] : r;
    }
    r = wave_min(r);
    if (lane_id() == 0) key[v] = ((v < first_star ? 1 : 2) << 22) | r;
}

// Locality of a layout: of a sample of instance rows (every kSample-th
// instance, kNearLanes lanes each), how many instance-to-instance entries
// lie within `near` execution rows of their row.  Each workgroup writes its
// counts (near, all) to part[2 b], part[2 b + 1].
constexpr int kNearLanes = 8;

__global__ void __launch_bounds__(kBT) k_near_count(int32_t n_inst, int32_t nearw, const int64_t* __restrict__ off,
                                                    const int32_t* __restrict__ len,
                                                    const int32_t* __restrict__ col, const int32_t* __restrict__ iperm,
                                                    int64_t* __restrict__ part) {
    __shared__ int64_t red[kBT / kWave];
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t v = (t / kNearLanes) * kSample;
    const int ln = threadIdx.x & (kNearLanes - 1);
    int64_t near = 0, all = 0;
    if (v < n_inst) {
        const int rv = iperm[v];
        const int64_t o = off[v];
        const int l = len[v];
        for (int j = ln; j < l; j += kNearLanes) {
            const int c = col[o + j];
            if (c >= n_inst) continue;
            const int d = iperm[c] - rv;
            near += (d <= nearw && d >= -nearw) ? 1 : 0;
            ++all;
        }
    }
    near = block_sum_i64<kBT>(near, red);
    all = block_sum_i64<kBT>(all, red);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = near;
        part[2 * blockIdx.x + 1] = all;
    }
}

// The verdict from the workgroups' counts: local when at least a quarter of
// the sampled entries are near their row (or nothing was sampled).
__global__ void __launch_bounds__(kBT) k_loc_flag(const int64_t* __restrict__ part, int32_t nparts,
                                                  int32_t* __restrict__ flag) {
    __shared__ int64_t red[kBT / kWave];
    int64_t near = 0, all = 0;
    for (int b = threadIdx.x; b < nparts; b += kBT) {
        near += part[2 * b];
        all += part[2 * b + 1];
    }
    near = block_sum_i64<kBT>(near, red);
    all = block_sum_i64<kBT>(all, red);
    if (threadIdx.x == 0) flag[0] = (all == 0 || 4 * near >= all) ? 1 : 0;
}

}  // namespace

static void exec_net_copy(Graph& g, int32_t N, hipStream_t s2);

// Two stable LSD passes over np keys (the low digit, then key >> lo_bits of
// that order) into `order`; ties keep node order.
static void sort_keys(Graph& g, const DevBuf<int32_t>& key, int32_t np, int lo_bits, int hi_bits,
                      DevBuf<int32_t>& order, hipStream_t s) {
    DevBuf<int32_t> first, sorted;
    sorted.ensure(static_cast<size_t>(np) + 1, s);
    SortKeys lo{key.p};
    lo.mask = (1 << lo_bits) - 1;
    lo.sorted = sorted.p;
    bucket_sort(g, lo, np, 1 << lo_bits, first, g.lay_start, s);
    SortKeys hi{sorted.p};
    hi.idx = first.p;
    hi.shift = lo_bits;
    hi.mask = (1 << hi_bits) - 1;
    bucket_sort(g, hi, np, 1 << hi_bits, order, g.lay_start, s);
    first.release(s);
    sorted.release(s);
}

// perm from the sorted order (instance windows by row length,
// macro pins and stars as sorted), then iperm.
static void finish_perm(Graph& g, const DevBuf<int32_t>& order, hipStream_t s) {
    const int32_t n = g.n_inst, N = g.n_tot, np = g.first_mvirt;
    g.perm.ensure(static_cast<size_t>(N) + 1, s);
    g.iperm.ensure(static_cast<size_t>(N) + 1, s);
    const unsigned windows = static_cast<unsigned>((n + kLenWindow - 1) / kLenWindow);
    const unsigned others = static_cast<unsigned>((N - n + kLenWindow - 1) / kLenWindow);
    if (windows + others)
        hipLaunchKernelGGL(k_window_sort, dim3(windows + others), dim3(kLenWindow), 0, s, n, np, N, order.p,
                           g.net_len.p, g.perm.p, g.iperm.p);
    AHR_LAUNCHED("k_window_sort");
}

// The Hilbert order of the placement's positions.
static void position_order(Graph& g, const float* pos, int32_t ncols, hipStream_t s) {
    const int32_t n = g.n_inst, np = g.first_mvirt;
    DevBuf<int32_t> key, order;
    key.ensure(static_cast<size_t>(np) + 1, s);
    const float side = static_cast<float>(1 << kGridBits);
    KeyArgs ka;
    ka.pos = pos;
    ka.ncols = ncols;
    ka.n_inst = n;
    ka.first_star = g.first_star;
    ka.first_mvirt = np;
    ka.mpin_pin = g.mpin_pin.p;
    ka.star_net = g.star_net.p;
    ka.net_ptr = g.nl.net_ptr;
    ka.pin_node = g.nl.pin_node;
    ka.pin_node_x = g.pin_node_x.p;
    ka.pin_off = g.nl.pin_off;
    ka.xl = g.nl.die[0];
    ka.yl = g.nl.die[1];
    ka.sx = side / (g.nl.die[2] - g.nl.die[0]);
    ka.sy = side / (g.nl.die[3] - g.nl.die[1]);
    hipLaunchKernelGGL(k_layout_keys, dim3(grid_for(np, kBT)), dim3(kBT), 0, s, ka, key.p);
    AHR_LAUNCHED("k_layout_keys");
    // the range bits keep the instances, macro pins and stars in their own id ranges
    sort_keys(g, key, np, kDigitBits, kKeyBits - kDigitBits, order, s);
    finish_perm(g, order, s);
    key.release(s);
    order.release(s);
}

// The locality test of the current layout, left on the device (g.loc_flag):
// of a sample of instance rows, the share of instance-to-instance entries
// within n/64 rows (at least 256) of their row.  g.hop_local is read later.
static void locality_begin(Graph& g, hipStream_t s) {
    const int32_t n = g.n_inst;
    const int64_t nt = (static_cast<int64_t>(n) + kSample - 1) / kSample;
    const unsigned blocks = grid_for(nt * kNearLanes, kBT);
    g.loc_part.ensure(2 * static_cast<size_t>(blocks), s);
    g.loc_flag.ensure(1, s);
    const int32_t nearw = n / 64 > 256 ? n / 64 : 256;
    hipLaunchKernelGGL(k_near_count, dim3(blocks), dim3(kBT), 0, s, n, nearw, g.net_off.p, g.net_len.p,
                       g.net_col.p, g.iperm.p, g.loc_part.p);
    AHR_LAUNCHED("k_near_count");
    hipLaunchKernelGGL(k_loc_flag, dim3(1), dim3(kBT), 0, s, g.loc_part.p, static_cast<int32_t>(blocks),
                       g.loc_flag.p);
    AHR_LAUNCHED("k_loc_flag");
    g.hop_local = -1;
}

// Whether the current layout's instance rows sit near their instance
// neighbours (the locality test, read now).
static bool layout_is_local(Graph& g, hipStream_t s) {
    locality_begin(g, s);
    int32_t f = 1;
    read_scalars({g.loc_flag.p}, &f, s);
    g.hop_local = f ? 1 : 0;
    return f != 0;
}

// Cuthill-McKee ranks of the instances (see the file's comment), then the
// netlist order of all instance, macro pin and star rows.
constexpr int kCmMaxLevels = 256;     // beyond that, the rest is appended in id order
constexpr int kCmCheck = 8;           // levels between reads of the level range

static void netlist_order(Graph& g, hipStream_t s) {
    const int32_t n = g.n_inst, np = g.first_mvirt;
    DevBuf<unsigned long long> lk;
    DevBuf<int32_t> rank, order, cnt, scn, bnd;
    const size_t n1 = static_cast<size_t>(n) + 1;
    lk.ensure(n1, s);
    rank.ensure(n1, s);
    order.ensure(n1, s);
    cnt.ensure(n1, s);
    scn.ensure(n1, s);
    bnd.ensure(4, s);
    g.scan_tmp.ensure(scan_tmp_elems(n), s);
    CmArgs a{n, g.net_off.p, g.net_len.p, g.net_col.p, lk.p, rank.p, order.p, cnt.p, scn.p, bnd.p};
    hipLaunchKernelGGL(k_cm_init, dim3(grid_for(n, kBT)), dim3(kBT), 0, s, a);
    AHR_LAUNCHED("k_cm_init");
    hipLaunchKernelGGL(k_cm_start, dim3(grid_for(n, kBT)), dim3(kBT), 0, s, a);
    AHR_LAUNCHED("k_cm_start");
    hipLaunchKernelGGL(k_cm_seed, dim3(1), dim3(1), 0, s, a);
    AHR_LAUNCHED("k_cm_seed");
    for (int k = 0; k < kCmMaxLevels; ++k) {
        hipLaunchKernelGGL(k_cm_expand, dim3(kCmGrid), dim3(256), 0, s, a, k);
        AHR_LAUNCHED("k_cm_expand");
        hipLaunchKernelGGL(k_cm_count, dim3(kCmGrid), dim3(256), 0, s, a, k);
        AHR_LAUNCHED("k_cm_count");
        scan_i32_to_i32(cnt.p, scn.p, n, g.scan_tmp.p, s);
        hipLaunchKernelGGL(k_cm_assign, dim3(kCmGrid), dim3(256), 0, s, a, k);
        AHR_LAUNCHED("k_cm_assign");
        hipLaunchKernelGGL(k_cm_next, dim3(1), dim3(1), 0, s, a);
        AHR_LAUNCHED("k_cm_next");
        if ((k + 1) % kCmCheck == 0) {
            int32_t lh[2];
            read_scalars({bnd.p, bnd.p + 1}, lh, s);
            if (lh[0] == lh[1]) break;
        }
    }
    // the unreached instances after the reached ones
    hipLaunchKernelGGL(k_cm_unplaced, dim3(grid_for(n, kBT)), dim3(kBT), 0, s, n, rank.p, cnt.p);
    AHR_LAUNCHED("k_cm_unplaced");
    scan_i32_to_i32(cnt.p, scn.p, n, g.scan_tmp.p, s);
    hipLaunchKernelGGL(k_cm_append, dim3(grid_for(n, kBT)), dim3(kBT), 0, s, n, cnt.p, scn.p, bnd.p, rank.p);
    AHR_LAUNCHED("k_cm_append");
    lk.release(s);
    order.release(s);
    cnt.release(s);
    scn.release(s);
    bnd.release(s);
    // sort keys: range, then rank (24 bits, two 12-bit passes)
    DevBuf<int32_t> skey, sorted;
    skey.ensure(static_cast<size_t>(np) + 1, s);
    hipLaunchKernelGGL(k_cm_keys, dim3(grid_for(n, kBT)), dim3(kBT), 0, s, n, rank.p, skey.p);
    AHR_LAUNCHED("k_cm_keys");
    if (np > n) {
        hipLaunchKernelGGL(k_cm_keys_aux, dim3(grid_for(static_cast<int64_t>(np - n) * kWave, kBT)), dim3(kBT), 0,
                           s, n, np, g.first_star, g.net_off.p, g.net_len.p, g.net_col.p, rank.p, skey.p);
        AHR_LAUNCHED("k_cm_keys_aux");
    }
    rank.release(s);
    sort_keys(g, skey, np, 12, 12, sorted, s);
    finish_perm(g, sorted, s);
    skey.release(s);
    sorted.release(s);
}

void set_layout(Graph& g, const float* pos, int32_t ncols, hipStream_t s) {
    const int32_t n = g.n_inst, N = g.n_tot, np = g.first_mvirt;
    const uint32_t fl = g.hp.flags;
    const bool cm_ok = n < (1 << 22);           // ranks fit the netlist order's 22-bit keys
    bool netlist = cm_ok && (fl & AHR_LAYOUT_NETLIST);
    bool tested = false;      // the locality test already covers the order taken
    if (!netlist) {
        position_order(g, pos, ncols, s);
        if (cm_ok && (fl & AHR_LAYOUT_AUTO)) {
            tested = layout_is_local(g, s);
            netlist = !tested;
        }
    }
    if (netlist) netlist_order(g, s);
    g.layout_netlist = netlist ? 1 : 0;
    // the hop's launch shape follows the order's locality (AHR_HOP_AUTO); the
    // verdict is read with the first row classes
    if (!tested) locality_begin(g, s);

    g.xqdeg.ensure(static_cast<size_t>(N) + 1, s);
    g.xmpin.ensure(static_cast<size_t>(g.first_star - n) + 1, s);
    g.xstar_net.ensure(static_cast<size_t>(np - g.first_star) + 1, s);
    g.xnet_rp.ensure(static_cast<size_t>(N) + 1, s);
    const bool hints = fl & (AHR_MACRO_HINTS | AHR_BIN_HINTS);
    if (hints) {
        g.xcell.ensure(static_cast<size_t>(n) + 1, s);
        g.xbase_w.ensure(static_cast<size_t>(n) + 1, s);
    }
    run_scans(scan_job(ExecRowScan{N, n, g.first_star, np, g.perm.p, g.net_len.p, g.qdeg.p, g.mpin_pin.p,
                                   g.nl.pin_node, g.nl.pin_off, g.star_net.p, g.nl.node_flags, g.nl.node_size,
                                   g.xqdeg.p, g.xmpin.p, g.xstar_net.p, hints ? g.xcell.p : nullptr, g.xbase_w.p,
                                   g.xnet_rp.p},
                       N),
              g.scan_tmp, s);
    g.xnet_ent.ensure(static_cast<size_t>(g.nnz_cap) + 1, s);      // the netlist arrays' bound
    if (g.nnz_cap) {
        // Nothing reads the execution-order entries before the first hop, so
        // their copy runs on the device's side stream, beside the hint build
        // and the degree kernels that follow on s.  Readers take the entries
        // through net_entries(), which orders their stream after the copy.
        if (!g.xnet_fork) AHR_HIP(hipEventCreateWithFlags(&g.xnet_fork, hipEventDisableTiming));
        if (!g.xnet_ready) AHR_HIP(hipEventCreateWithFlags(&g.xnet_ready, hipEventDisableTiming));
        const hipStream_t s2 = side_stream();
        AHR_HIP(hipEventRecord(g.xnet_fork, s));
        AHR_HIP(hipStreamWaitEvent(s2, g.xnet_fork, 0));
        try {
            exec_net_copy(g, N, s2);
        } catch (...) {
            // readers and the destructor still order themselves after what
            // did reach the side stream
            (void)hipEventRecord(g.xnet_ready, s2);
            throw;
        }
        AHR_HIP(hipEventRecord(g.xnet_ready, s2));
        g.xnet_waited = 0;
    }
    g.has_layout = 1;
}

// The execution-order netlist entries: short rows by k_exec_net, long rows
// by k_exec_net_long, all on stream s2.
static void exec_net_copy(Graph& g, int32_t N, hipStream_t s2) {
    hipLaunchKernelGGL(k_exec_net, dim3(xcd_grid(grid_for(N, kExecRows))), dim3(kBT), 0, s2, N,
                       g.perm.p, g.iperm.p, g.net_off.p, g.net_col.p, g.net_q.p, g.xnet_rp.p, g.xnet_ent.p);
    AHR_LAUNCHED("k_exec_net");
    if (g.n_long_nodes) {
        hipLaunchKernelGGL(k_exec_net_long, dim3(g.n_long_nodes), dim3(kBT), 0, s2, g.long_nodes.p, g.iperm.p,
                           g.net_off.p, g.net_col.p, g.net_q.p, g.xnet_rp.p, g.xnet_ent.p);
        AHR_LAUNCHED("k_exec_net_long");
    }
}

const int2* net_entries(const Graph& g, hipStream_t s) {
    if (g.xnet_ready && !(g.xnet_waited && g.xnet_wait_stream == s)) {
        AHR_HIP(hipStreamWaitEvent(s, g.xnet_ready, 0));
        g.xnet_waited = 1;
        g.xnet_wait_stream = s;
    }
    return g.xnet_ent.p;
}

}  // namespace ahr
