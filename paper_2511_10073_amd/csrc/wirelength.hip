// Weighted-average (WA) wirelength and its gradient (Section II-B of the
// paper, "Wirelength model"): for each net and axis the exponentially
// weighted means of the pin coordinates with weights exp(+x/gamma) (smooth
// maximum) and exp(-x/gamma) (smooth minimum); W sums their differences over
// nets and both axes.  This is the wirelength term of the electrostatic
// global placer that consumes the initializer's placement.
//
// Numbers: coordinates, sums and ratios in float64; each weight is taken
// relative to the net's extreme coordinate (exp((x - max)/gamma),
// exp((min - x)/gamma), which cancels in every ratio) and exponentiated in
// float32 (arguments <= 0, values in (0, 1], relative error ~1e-7): the
// weights are what the placer's gradient step needs, and float64
// exponentials cost the pass several times its memory time.  Gradient of pin i:
//   p+_i (1 + (x_i - xbar+)/gamma) - p-_i (1 - (x_i - xbar-)/gamma),
// p+-_i the pin's normalised weight.  An instance's gradient is the sum over
// its pins, added in int64 fixed point (2^-40 units), so the order in which
// the node pass meets the pins does not change the result.
//
// Layout: an index built once per netlist (ahr_wl_create) gives every pin its
// place among the pins ordered by instance (node_ptr / place) and lists the
// nets of more than 64 pins.  One call is three kernels: the net pass (256
// nets a workgroup, and one workgroup for each net of more than 64 pins),
// writing net totals into workgroup partials and every pin's gradient to its
// place in a [pins][ncols] float64 buffer; the node pass (one thread per
// instance reads its pins' consecutive rows); and the fixed-order reduction
// of the partials.  The net pass scatters and the node pass streams, as a
// store in flight holds up no wave: with the buffer in pin order and the node
// pass gathering, the two take 278 + 225 us at 2.2M cells and 2 columns,
// against 410 + 69 us this way.
#include <cmath>

#include "ahr_internal.hpp"
#include "device_util.hpp"
#include "scan.hpp"

namespace ahr {

namespace {

constexpr int kBT = 256;
constexpr int kMaxPairs = 4;
constexpr double kFix = 1099511627776.0;          // 2^40
constexpr double kUnfix = 1.0 / 1099511627776.0;

struct WlIndex {
    ahr_netlist nl;
    DevBuf<int32_t> node_ptr;     // [n_inst + 1]
    DevBuf<int32_t> place;        // [n_pins] where each pin's gradient goes: instances ascending (pins of one in no order)
    DevBuf<int32_t> big;          // nets of more than kWave pins, ascending
    int32_t n_big = 0;
    int device = 0;
    mutable hipStream_t work_stream = nullptr;
    mutable int stream_uses = 0;
    void use_stream(hipStream_t s) const {
        if (stream_uses == 0) {
            work_stream = s;
            stream_uses = 1;
        } else if (s != work_stream) {
            stream_uses = 2;
        }
    }
    ~WlIndex() {
        hipStream_t s = stream_uses == 1 ? work_stream : nullptr;
        if (stream_uses > 1) (void)hipDeviceSynchronize();
        node_ptr.release(s);
        place.release(s);
        big.release(s);
    }
};

// The nets of more than kWave pins, ascending.
struct BigNetScan {
    static constexpr int K = 1;
    static constexpr bool kTotal = false, kHeavy = false;
    using Raw = Pack<1>;
    __device__ Pack<1> pack(const Pack<1>& p) const { return p; }
    const int32_t* net_ptr;
    int32_t* list;              // or null: count only
    int32_t* count;
    __device__ Pack<1> first(int64_t e) const { return {{net_ptr[e + 1] - net_ptr[e] > kWave ? 1 : 0}}; }
    __device__ Pack<1> again(int64_t e) const { return first(e); }
    __device__ void item(int64_t e, const Pack<1>& own, const Pack<1>& before, const Pack<1>&) const {
        if (list && own.v[0]) list[before.v[0]] = static_cast<int32_t>(e);
    }
    __device__ void done(const Pack<1>& total) const { *count = static_cast<int32_t>(total.v[0]); }
};

__global__ void k_pin_slots(const int32_t* __restrict__ pin_node, int32_t n_pins, int32_t* __restrict__ cnt,
                            int32_t* __restrict__ slot) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p < n_pins) slot[p] = atomicAdd(&cnt[pin_node[p]], 1);
}

__global__ void k_pin_places(const int32_t* __restrict__ pin_node, int32_t n_pins,
                             const int32_t* __restrict__ node_ptr, int32_t* __restrict__ slot) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p < n_pins) slot[p] += node_ptr[pin_node[p]];
}

// exp(a) for a <= 0, in float32.
__device__ __forceinline__ double wexp(double a) { return static_cast<double>(expf(static_cast<float>(a))); }

// One net's sums in one column.
struct ColAcc {
    double hi, lo;      // extremes
    double sp, tp;      // sum exp((x-hi)/g), sum x exp((x-hi)/g)
    double sm, tm;      // sum exp((lo-x)/g), sum x exp((lo-x)/g)
};

__device__ __forceinline__ double gpin(double x, const ColAcc& a, double inv_g) {
    const double xp = a.tp / a.sp, xm = a.tm / a.sm;
    const double pp = wexp((x - a.hi) * inv_g) / a.sp, pm = wexp((a.lo - x) * inv_g) / a.sm;
    return pp * (1.0 + (x - xp) * inv_g) - pm * (1.0 - (x - xm) * inv_g);
}

// One row of C float32 coordinates.
template <int C>
__device__ __forceinline__ void load_row(const float* p, float* v) {
    if constexpr (C == 2) {
        const float2 t = *reinterpret_cast<const float2*>(p);
        v[0] = t.x;
        v[1] = t.y;
    } else {
#pragma unroll
        for (int h = 0; h < C / 4; ++h) {
            const float4 t = reinterpret_cast<const float4*>(p)[h];
            v[4 * h] = t.x;
            v[4 * h + 1] = t.y;
            v[4 * h + 2] = t.z;
            v[4 * h + 3] = t.w;
        }
    }
}

// Coordinate in column c of a pin: its instance's position + its offset (x or y).
__device__ __forceinline__ double coord(const float (&v), float2 off, int c) {
    return static_cast<double>(v) + static_cast<double>((c & 1) ? off.y : off.x);
}

// One net by one thread, a column at a time.
template <int P>
__device__ __forceinline__ void wa_alone(const float* __restrict__ pos, const int32_t* __restrict__ pin_node,
                                         const float* __restrict__ pin_off, int p0, int p1, double inv_g, double* tot,
                                         const int32_t* __restrict__ place, double* __restrict__ pin_g) {
    constexpr int C = 2 * P;
#pragma unroll 1
    for (int c = 0; c < C; ++c) {
        const auto at = [&](int p) {
            return static_cast<double>(pos[static_cast<int64_t>(pin_node[p]) * C + c]) +
                   static_cast<double>(pin_off[2 * p + (c & 1)]);
        };
        ColAcc a{-1e300, 1e300, 0, 0, 0, 0};
#pragma unroll 1
        for (int p = p0; p < p1; ++p) {
            const double x = at(p);
            a.hi = __builtin_fmax(a.hi, x);
            a.lo = __builtin_fmin(a.lo, x);
        }
#pragma unroll 1
        for (int p = p0; p < p1; ++p) {
            const double x = at(p), f = wexp((x - a.hi) * inv_g), h = wexp((a.lo - x) * inv_g);
            a.sp += f;
            a.tp += x * f;
            a.sm += h;
            a.tm += x * h;
        }
        const double w = a.tp / a.sp - a.tm / a.sm;
#pragma unroll
        for (int q = 0; q < P; ++q) tot[q] += q == c / 2 ? w : 0.0;
        if (!pin_g) continue;
#pragma unroll 1
        for (int p = p0; p < p1; ++p) pin_g[static_cast<int64_t>(place[p]) * C + c] = gpin(at(p), a, inv_g);
    }
}

// The nets of up to kWave pins, kBT of them a workgroup.  Their pins are
// consecutive, so they are read with one lane a pin (coalesced node and offset
// loads, every gather in flight) in runs of whole nets of at most kRun pins;
// each column pair's coordinates go to LDS, and the work alternates between
// one thread a net (extremes, then the shifted sums in pin order) and one lane
// a pin (the two weights, then the gradient), so the exponentials and the
// stores idle no lane and every weight is taken once.  Pins of larger nets
// are left out.
//
// What bounds it: the position gathers (HPWL, which makes the same ones, takes
// 134 us at 1.1M cells) and the scattered stores of the gradient, with the
// waves in flight, which LDS and registers limit: the nets' extremes lie where
// the weights then go, and the means where the coordinates were, so that four
// workgroups fit a CU instead of three, and the large nets beside the batches
// take a few column pairs at a time.  A net's thread reads a pin with two
// 16-byte reads and several pins at once: in arrays an axis, a pin after
// another, its loops were the longest part of a small netlist's call (7,000
// cells, 8 columns: 133 us for 101, 105 for 72 without the gradient).
// Against one thread a net, over nets sorted by size, with the pins in
// registers and the gradients in pin order, a call takes, at 2.2M cells and 2,
// 4 and 8 columns, 436, 626 and 1206 us for 792, 956 and 1348, without the
// gradient 189, 310 and 604 for 368, 420 and 535; at 2,000 cells 48, 74 and 123
// for 82, 119 and 194, without it 25, 38 and 71 for 28, 40 and 65.
constexpr int kRun = 1024;
constexpr int kMaxPins = 4;                             // pins whose coordinates a thread reads at a time for the extremes
template <int P, bool Grad>
constexpr int kSumPins = Grad && P > 1 ? 2 : 4;         // and for the sums: more take registers of the gradient's waves

template <int P, bool Grad>
__device__ __forceinline__ void wa_batch(const float* __restrict__ pos, const int32_t* __restrict__ net_ptr,
                                         int32_t n_nets, int32_t batch, const int32_t* __restrict__ pin_node,
                                         const float* __restrict__ pin_off, double inv_g, double* tot,
                                         const int32_t* __restrict__ place, double* __restrict__ pin_g) {
    constexpr int C = 2 * P, U = kRun / kBT, S = kSumPins<P, Grad>;
    static_assert(kRun >= 4 * kBT, "a run's coordinates leave room for the nets' means");
    __shared__ double2 xy[kRun];                // a pair's coordinates; then [mean, reciprocal sum] of each net
    __shared__ float4 ew[kRun];                 // the weights (x max, x min, y max, y min); before, each net's extremes
    double2* ex = reinterpret_cast<double2*>(ew);
    __shared__ uint8_t owner[kRun];
    __shared__ int bstart[kBT], blen[kBT], cnt[kBT / kWave], stop_q[2], down;
    const int t = threadIdx.x;
    if (t == 0) down = 0;
    const int64_t c0 = static_cast<int64_t>(batch) * kBT, e = c0 + t;
    const int64_t last = c0 + kBT < n_nets ? c0 + kBT : n_nets;
    const int first = net_ptr[c0];
    const int p0 = net_ptr[e < last ? e : last], p1 = net_ptr[e < last ? e + 1 : last];
    const bool big = p1 - p0 > kWave;
    int nb;
    const int k = block_rank<kBT>(big, cnt, &nb);      // (its barriers follow down = 0)
    if (big) {
        bstart[k] = p0;
        blen[k] = p1 - p0;
    }
    if (p1 < p0) down = 1;
    __syncthreads();
    // A net_ptr that decreases is no netlist, but the host has not seen it: the
    // count of the pins below might not end, or leave the nets' ranges.
    if (down) {
        if (p1 > p0 && !big) wa_alone<P>(pos, pin_node, pin_off, p0, p1, inv_g, tot, place, pin_g);
        return;
    }
    // the pins without the big nets' are counted from 0; pins of big nets
    // before place q of that count
    auto shift = [&](int q) {
        int sh = 0;
        for (int b = 0; b < nb && bstart[b] - first - sh <= q; ++b) sh += blen[b];
        return sh;
    };
    int skipped = 0, all = 0;
    for (int b = 0; b < nb; ++b) {
        skipped += bstart[b] < p0 ? blen[b] : 0;
        all += blen[b];
    }
    const int n = net_ptr[last] - first - all;
    const int q0 = p0 - first - skipped, q1 = big ? q0 : q0 + (p1 - p0);
    for (int at = 0, run = 0; at < n; ++run) {
        // the run: the nets from place `at` on that end within kRun pins
        const bool in_run = q0 >= at && q1 > q0 && q1 <= at + kRun;
        if (t == 0) stop_q[run & 1] = at;
        __syncthreads();
        if (in_run) atomicMax(&stop_q[run & 1], q1);
        __syncthreads();
        const int m = stop_q[run & 1] - at;        // at least one net's pins
        int v[U], pin[U];
        int at_g[U];
        float2 off[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = at + (t + u * kBT < m ? t + u * kBT : m - 1);
            pin[u] = first + q + shift(q);
            v[u] = pin_node[pin[u]];
            off[u] = reinterpret_cast<const float2*>(pin_off)[pin[u]];
            at_g[u] = Grad ? place[pin[u]] : 0;
        }
        float g[U][C];
#pragma unroll
        for (int u = 0; u < U; ++u) load_row<C>(pos + static_cast<int64_t>(v[u]) * C, g[u]);
        const int a = q0 - at, b = q1 - at;        // this thread's net inside the run
        for (int pr = 0; pr < P; ++pr) {
            double2 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float gx = g[u][0], gy = g[u][1];
#pragma unroll
                for (int q = 1; q < P; ++q) {
                    gx = pr == q ? g[u][2 * q] : gx;
                    gy = pr == q ? g[u][2 * q + 1] : gy;
                }
                x[u] = make_double2(coord(gx, off[u], 0), coord(gy, off[u], 1));
                xy[t + u * kBT] = x[u];
            }
            __syncthreads();
            if (in_run) {
                double2 hi = {-1e300, -1e300}, lo = {1e300, 1e300};
                for (int i = a; i < b; i += kMaxPins) {           // kMaxPins pins' reads at once (the last one repeats)
                    double2 y[kMaxPins];
#pragma unroll
                    for (int u = 0; u < kMaxPins; ++u) {
                        const int j = i + u < b ? i + u : b - 1;
                        if (pr == 0) owner[j] = static_cast<uint8_t>(t);
                        y[u] = xy[j];
                    }
#pragma unroll
                    for (int u = 0; u < kMaxPins; ++u) {
                        hi.x = __builtin_fmax(hi.x, y[u].x);
                        lo.x = __builtin_fmin(lo.x, y[u].x);
                        hi.y = __builtin_fmax(hi.y, y[u].y);
                        lo.y = __builtin_fmin(lo.y, y[u].y);
                    }
                }
                ex[2 * t] = make_double2(hi.x, lo.x);
                ex[2 * t + 1] = make_double2(hi.y, lo.y);
            }
            __syncthreads();
            float4 w[U];
            int own[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                own[u] = owner[t + u * kBT < m ? t + u * kBT : m - 1];
                const double2 ax = ex[2 * own[u]], ay = ex[2 * own[u] + 1];
                w[u].x = expf(static_cast<float>((x[u].x - ax.x) * inv_g));
                w[u].y = expf(static_cast<float>((ax.y - x[u].x) * inv_g));
                w[u].z = expf(static_cast<float>((x[u].y - ay.x) * inv_g));
                w[u].w = expf(static_cast<float>((ay.y - x[u].y) * inv_g));
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) ew[t + u * kBT] = w[u];
            __syncthreads();
            double2 sp = {0, 0}, tp = {0, 0}, sm = {0, 0}, tm = {0, 0};
            if (in_run) {
                const auto add = [&](const double2& y, const float4& f) {
                    sp.x += f.x;
                    tp.x += y.x * f.x;
                    sm.x += f.y;
                    tm.x += y.x * f.y;
                    sp.y += f.z;
                    tp.y += y.y * f.z;
                    sm.y += f.w;
                    tm.y += y.y * f.w;
                };
                int i = a;
#pragma unroll 1
                for (; i + S <= b; i += S) {               // S pins' reads at once, added in order
                    double2 y[S];
                    float4 f[S];
#pragma unroll
                    for (int u = 0; u < S; ++u) {
                        y[u] = xy[i + u];
                        f[u] = ew[i + u];
                    }
#pragma unroll
                    for (int u = 0; u < S; ++u) add(y[u], f[u]);
                }
#pragma unroll 1
                for (; i < b; ++i) add(xy[i], ew[i]);
                const double wa = (0.0 + (tp.x / sp.x - tm.x / sm.x)) + (tp.y / sp.y - tm.y / sm.y);
#pragma unroll
                for (int q = 0; q < P; ++q) tot[q] += pr == q ? wa : 0.0;
            }
            __syncthreads();
            if constexpr (!Grad) continue;
            if (in_run) {
                const double2 rp = {1.0 / sp.x, 1.0 / sp.y}, rm = {1.0 / sm.x, 1.0 / sm.y};
                xy[4 * t] = make_double2(rp.x, rm.x);
                xy[4 * t + 1] = make_double2(tp.x * rp.x, tm.x * rm.x);
                xy[4 * t + 2] = make_double2(rp.y, rm.y);
                xy[4 * t + 3] = make_double2(tp.y * rp.y, tm.y * rm.y);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const auto d = [&](double y, float fp, float fm, const double2& r, const double2& mean) {
                    const double pp = static_cast<double>(fp) * r.x, pm = static_cast<double>(fm) * r.y;
                    return pp * (1.0 + (y - mean.x) * inv_g) - pm * (1.0 - (y - mean.y) * inv_g);
                };
                const double2* net = xy + 4 * own[u];
                const double dx = d(x[u].x, w[u].x, w[u].y, net[0], net[1]), dy = d(x[u].y, w[u].z, w[u].w, net[2], net[3]);
                if (t + u * kBT < m)
                    *reinterpret_cast<double2*>(pin_g + static_cast<int64_t>(at_g[u]) * C + 2 * pr) = make_double2(dx, dy);
            }
            __syncthreads();
        }
        at += m;
    }
}

// Running (shifted) exponential sums: value m (the shift: the largest x so
// far for the maximum side, the smallest for the minimum side), sum of
// exp(+-(x - m)/g) and of x times it; merging rescales the side with the
// smaller (larger) shift.  One pass gives what the three-pass form gives.
struct Run {
    double m, s, t;
};

__device__ __forceinline__ void run_add(Run& r, double x, double sgn_inv_g) {
    // sgn_inv_g = +1/g (maximum side) or -1/g (minimum side)
    const double q = (x - r.m) * sgn_inv_g;
    if (q > 0) {            // new extreme: rescale what is there
        const double f = wexp(-q);
        r.s = r.s * f + 1.0;
        r.t = r.t * f + x;
        r.m = x;
    } else {
        const double e = wexp(q);
        r.s += e;
        r.t += x * e;
    }
}

__device__ __forceinline__ Run run_merge(Run a, Run b, double sgn_inv_g) {
    if (b.s == 0) return a;
    if (a.s == 0) return b;
    if ((b.m - a.m) * sgn_inv_g > 0) {
        Run t = a;
        a = b;
        b = t;
    }
    const double f = wexp((b.m - a.m) * sgn_inv_g);
    return Run{a.m, a.s + b.s * f, a.t + b.t * f};
}

// A net above kWave pins by one workgroup: one pass for the shifted sums of
// every column, one for the gradients, kBigU pins a lane in flight.
constexpr int kBigU = 4;

// The lane's pins p, p + kBT, ... (clamped to the net's last): rows and offsets.
template <int C, int S>
__device__ __forceinline__ void big_pins(const float* __restrict__ pos, const int32_t* __restrict__ pin_node,
                                         const float* __restrict__ pin_off, int p, int p1, float (&v)[kBigU][C],
                                         float2 (&off)[kBigU]) {
    int node[kBigU];
#pragma unroll
    for (int u = 0; u < kBigU; ++u) {
        const int q = p + u * kBT < p1 ? p + u * kBT : p1 - 1;
        node[u] = pin_node[q];
        off[u] = reinterpret_cast<const float2*>(pin_off)[q];
    }
#pragma unroll
    for (int u = 0; u < kBigU; ++u) load_row<C>(pos + static_cast<int64_t>(node[u]) * S, v[u]);
}

// P column pairs of rows of S columns.
template <int P, int S>
__device__ __forceinline__ void wa_big(const float* __restrict__ pos, const int32_t* __restrict__ pin_node,
                                       const float* __restrict__ pin_off, int p0, int p1, double inv_g, double* tot,
                                       const int32_t* __restrict__ place, double* __restrict__ pin_g) {
    constexpr int C = 2 * P;
    __shared__ Run red[C][2][kBT / kWave];
    Run rp[C], rm[C];
    float v[kBigU][C];
    float2 off[kBigU];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        rp[c] = Run{-1e300, 0, 0};
        rm[c] = Run{1e300, 0, 0};
    }
    for (int p = p0 + threadIdx.x; p < p1; p += kBigU * kBT) {
        big_pins<C, S>(pos, pin_node, pin_off, p, p1, v, off);
#pragma unroll
        for (int u = 0; u < kBigU; ++u) {
            if (p + u * kBT >= p1) break;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const double x = coord(v[u][c], off[u], c);
                if (rp[c].s == 0) {
                    rp[c] = Run{x, 1.0, x};
                    rm[c] = Run{x, 1.0, x};
                } else {
                    run_add(rp[c], x, inv_g);
                    run_add(rm[c], x, -inv_g);
                }
            }
        }
    }
    // wave then workgroup merges, in a fixed order
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            Run a{__shfl_xor(rp[c].m, o), __shfl_xor(rp[c].s, o), __shfl_xor(rp[c].t, o)};
            Run b{__shfl_xor(rm[c].m, o), __shfl_xor(rm[c].s, o), __shfl_xor(rm[c].t, o)};
            // lane pairs merge in lane order so both lanes hold the same bits
            rp[c] = (lane_id() & o) ? run_merge(a, rp[c], inv_g) : run_merge(rp[c], a, inv_g);
            rm[c] = (lane_id() & o) ? run_merge(b, rm[c], -inv_g) : run_merge(rm[c], b, -inv_g);
        }
        if (lane_id() == 0) {
            red[c][0][wave_id()] = rp[c];
            red[c][1][wave_id()] = rm[c];
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) {
        rp[c] = red[c][0][0];
        rm[c] = red[c][1][0];
        for (int w = 1; w < kBT / kWave; ++w) {
            rp[c] = run_merge(rp[c], red[c][0][w], inv_g);
            rm[c] = run_merge(rm[c], red[c][1][w], -inv_g);
        }
    }
    if (pin_g) {
        for (int p = p0 + threadIdx.x; p < p1; p += kBigU * kBT) {
            big_pins<C, S>(pos, pin_node, pin_off, p, p1, v, off);
#pragma unroll
            for (int u = 0; u < kBigU; ++u) {
                if (p + u * kBT >= p1) break;
                const int64_t k = static_cast<int64_t>(place[p + u * kBT]) * S;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const ColAcc a{rp[c].m, rm[c].m, rp[c].s, rp[c].t, rm[c].s, rm[c].t};
                    pin_g[k + c] = gpin(coord(v[u][c], off[u], c), a, inv_g);
                }
            }
        }
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < P; ++c)
            tot[c] = (rp[2 * c].t / rp[2 * c].s - rm[2 * c].t / rm[2 * c].s) +
                     (rp[2 * c + 1].t / rp[2 * c + 1].s - rm[2 * c + 1].t / rm[2 * c + 1].s);
    }
}

// The net pass: workgroups [0, n_big) take a large net each (first, as the
// longest of them outlast a batch), the others a batch of kBT nets.
// Workgroup totals to partial[blockIdx.x].
template <int P, bool Grad>
__global__ void __launch_bounds__(kBT, P == 4 && Grad ? 1 : 4)
    k_wa_nets(const float* __restrict__ pos, const int32_t* __restrict__ net_ptr, int32_t n_nets,
              const int32_t* __restrict__ big, int32_t n_big, const int32_t* __restrict__ pin_node,
              const float* __restrict__ pin_off, double inv_g, double* __restrict__ partial,
              const int32_t* __restrict__ place, double* __restrict__ pin_g) {
    __shared__ double red[kBT / kWave];
    double tot[P];
#pragma unroll
    for (int q = 0; q < P; ++q) tot[q] = 0;
    const int32_t blk = static_cast<int32_t>(blockIdx.x);
    if (blk < n_big) {
        const int e = big[blk];
        // a few column pairs at a time: all four at once take 233 registers, and the
        // batches beside them run at two waves a SIMD
        constexpr int T = P < 4 ? P : Grad ? 2 : 1;
#pragma unroll 1
        for (int q = 0; q < P; q += T) {
            if (q) __syncthreads();
            double part[T] = {};
            wa_big<T, 2 * P>(pos + 2 * q, pin_node, pin_off, net_ptr[e], net_ptr[e + 1], inv_g, part, place,
                             Grad ? pin_g + 2 * q : nullptr);
#pragma unroll
            for (int c = 0; c < P; ++c)
#pragma unroll
                for (int d = 0; d < T; ++d) tot[c] = c == q + d ? part[d] : tot[c];
        }
    } else {
        wa_batch<P, Grad>(pos, net_ptr, n_nets, blk - n_big, pin_node, pin_off, inv_g, tot, place, pin_g);
    }
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const double s = block_sum_f64<kBT>(tot[q], red);
        if (threadIdx.x == 0) partial[static_cast<int64_t>(blk) * kMaxPairs + q] = s;
    }
}

// Gradient of every instance: the exact (int64, 2^-40 units) sum of its
// pins' gradients, rounded once to float32.
template <int C>
__global__ void __launch_bounds__(kBT) k_wa_nodes(const int32_t* __restrict__ node_ptr,
                                                  const double* __restrict__ pin_g, int32_t n_inst,
                                                  float* __restrict__ grad) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * kBT + threadIdx.x;
    if (v >= n_inst) return;
    long long acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0;
    const int k0 = node_ptr[v], k1 = node_ptr[v + 1];
    // kB pins at a time, every load in flight (indexes clamped to the last
    // pin; the repeats are not added)
    constexpr int kB = 4;
    for (int b = k0; b < k1; b += kB) {
        double g[kB][C];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const double2* r =
                reinterpret_cast<const double2*>(pin_g + static_cast<int64_t>(b + u < k1 ? b + u : k1 - 1) * C);
#pragma unroll
            for (int h = 0; h < C / 2; ++h) {
                const double2 t = r[h];
                g[u][2 * h] = t.x;
                g[u][2 * h + 1] = t.y;
            }
        }
#pragma unroll
        for (int u = 0; u < kB; ++u)
            if (b + u < k1)
#pragma unroll
                for (int c = 0; c < C; ++c) acc[c] += llrint(g[u][c] * kFix);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) grad[v * C + c] = static_cast<float>(static_cast<double>(acc[c]) * kUnfix);
}

constexpr int kFinalBT = 1024;

// The partials in a fixed order: thread t adds partials t, t + kFinalBT, ...
// in turn, then a fixed block reduction.
__global__ void __launch_bounds__(kFinalBT) k_wa_final(const double* __restrict__ partial, int nparts, int npairs,
                                                       double* __restrict__ out) {
    __shared__ double red[kFinalBT / kWave];
    for (int c = 0; c < npairs; ++c) {
        double s = 0;
        for (int b = threadIdx.x; b < nparts; b += kFinalBT) s += partial[static_cast<int64_t>(b) * kMaxPairs + c];
        s = block_sum_f64<kFinalBT>(s, red);
        if (threadIdx.x == 0) out[c] = s;
    }
}

template <int P>
void wa_p(const WlIndex& w, const float* pos, double inv_g, double* wl, float* grad, hipStream_t s) {
    const ahr_netlist& nl = w.nl;
    constexpr int C = 2 * P;
    const int grid = w.n_big + static_cast<int>((static_cast<int64_t>(nl.n_nets) + kBT - 1) / kBT);
    DevBuf<double> partial, pin_g;
    partial.ensure(static_cast<size_t>(grid + 1) * kMaxPairs, s);
    if (grad) pin_g.ensure(static_cast<size_t>(nl.n_pins > 0 ? nl.n_pins : 1) * C, s);
    const double bytes = static_cast<double>(nl.n_pins) * (4 + 8 + 4 * C + (grad ? 8 * C * 2 + 4 : 0)) +
                         static_cast<double>(nl.n_nets + 1) * 4 +
                         (grad ? static_cast<double>(nl.n_inst) * (4 + 4 * C) : 0.0);
    {
        ProfScope ps(kStageWa, s, bytes);
        if (grid) {
            hipLaunchKernelGGL((grad ? k_wa_nets<P, true> : k_wa_nets<P, false>), dim3(grid), dim3(kBT), 0, s, pos,
                               nl.net_ptr, nl.n_nets, w.big.p, w.n_big, nl.pin_node, nl.pin_off, inv_g, partial.p,
                               w.place.p, grad ? pin_g.p : nullptr);
            AHR_LAUNCHED("k_wa_nets");
        }
        if (grad) {
            hipLaunchKernelGGL(k_wa_nodes<C>, dim3(grid_for(nl.n_inst, kBT)), dim3(kBT), 0, s, w.node_ptr.p,
                               pin_g.p, nl.n_inst, grad);
            AHR_LAUNCHED("k_wa_nodes");
        }
        hipLaunchKernelGGL(k_wa_final, dim3(1), dim3(kFinalBT), 0, s, partial.p, grid, P, wl);
        AHR_LAUNCHED("k_wa_final");
    }
    partial.release(s);
    pin_g.release(s);
}

}  // namespace

}  // namespace ahr

using ahr::fail;

extern "C" {

ahr_status ahr_wl_create(const ahr_netlist* nl, void* stream, ahr_wl** out) {
    if (!nl) return fail(AHR_EINVAL, "netlist is NULL");
    if (!out) return fail(AHR_EINVAL, "out is NULL");
    if (nl->n_inst <= 0 || nl->n_nets < 0 || nl->n_pins < 0 || nl->reserved0 != 0 || !nl->net_ptr ||
        (nl->n_pins > 0 && (!nl->pin_node || !nl->pin_off)))
        return fail(AHR_EINVAL, "bad netlist (counts, reserved0 or NULL arrays)");
    try {
        ahr::set_error(AHR_OK, "");
        hipStream_t s = static_cast<hipStream_t>(stream);
        auto* w = new ahr::WlIndex();
        w->nl = *nl;
        w->use_stream(s);
        try {
            AHR_HIP(hipGetDevice(&w->device));
            const int32_t n = nl->n_inst, P = nl->n_pins;
            ahr::DevBuf<int32_t> cnt;
            ahr::DevBuf<int64_t> tmp;
            cnt.ensure(static_cast<size_t>(n) + 1, s);
            tmp.ensure(ahr::scan_tmp_elems(n), s);
            w->node_ptr.ensure(static_cast<size_t>(n) + 1, s);
            w->place.ensure(static_cast<size_t>(P > 0 ? P : 1), s);
            ahr::fill_i32(cnt.p, n, 0, s);
            if (P > 0) {
                hipLaunchKernelGGL(ahr::k_pin_slots, dim3(ahr::grid_for(P, ahr::kBT)), dim3(ahr::kBT), 0, s,
                                   nl->pin_node, P, cnt.p, w->place.p);
                AHR_LAUNCHED("k_pin_slots");
            }
            ahr::scan_i32_to_i32(cnt.p, w->node_ptr.p, n, tmp.p, s);
            if (P > 0) {
                hipLaunchKernelGGL(ahr::k_pin_places, dim3(ahr::grid_for(P, ahr::kBT)), dim3(ahr::kBT), 0, s,
                                   nl->pin_node, P, w->node_ptr.p, w->place.p);
                AHR_LAUNCHED("k_pin_places");
            }
            // nets above kWave pins, ascending: counted, then listed
            if (nl->n_nets > 0) {
                ahr::DevBuf<int32_t> count;
                count.ensure(1, s);
                ahr::run_scans(ahr::scan_job(ahr::BigNetScan{nl->net_ptr, nullptr, count.p}, nl->n_nets), tmp, s);
                w->n_big = ahr::read_i32(count.p, s);
                w->big.ensure(static_cast<size_t>(w->n_big) + 1, s);
                if (w->n_big)
                    ahr::run_scans(ahr::scan_job(ahr::BigNetScan{nl->net_ptr, w->big.p, count.p}, nl->n_nets), tmp, s);
                count.release(s);
            }
            cnt.release(s);
            tmp.release(s);
            AHR_HIP(hipStreamSynchronize(s));
        } catch (...) {
            delete w;
            throw;
        }
        *out = reinterpret_cast<ahr_wl*>(w);
        ahr::flush_frees();
        return AHR_OK;
    } catch (const ahr::Error& e) {
        ahr::flush_frees();
        return fail(e.code, e.msg);
    } catch (...) {
        ahr::flush_frees();
        return fail(AHR_EDEVICE, "unexpected exception");
    }
}

ahr_status ahr_wa(ahr_wl* h, const float* g, int32_t ncols, float gamma, double* wl, float* grad, void* stream) {
    if (!h) return fail(AHR_EINVAL, "wirelength index is NULL");
    if (!g || !wl) return fail(AHR_EINVAL, "g/wl is NULL");
    if (ncols != 2 && ncols != 4 && ncols != 8) return fail(AHR_EINVAL, "ncols must be 2, 4 or 8");
    if (!(gamma > 0.f) || !std::isfinite(gamma)) return fail(AHR_EINVAL, "gamma must be positive and finite");
    try {
        ahr::set_error(AHR_OK, "");
        const auto* w = reinterpret_cast<const ahr::WlIndex*>(h);
        hipStream_t s = static_cast<hipStream_t>(stream);
        w->use_stream(s);
        const double inv_g = 1.0 / static_cast<double>(gamma);
        switch (ncols) {
            case 2: ahr::wa_p<1>(*w, g, inv_g, wl, grad, s); break;
            case 4: ahr::wa_p<2>(*w, g, inv_g, wl, grad, s); break;
            default: ahr::wa_p<4>(*w, g, inv_g, wl, grad, s); break;
        }
        ahr::flush_frees();
        return AHR_OK;
    } catch (const ahr::Error& e) {
        ahr::flush_frees();
        return fail(e.code, e.msg);
    } catch (...) {
        ahr::flush_frees();
        return fail(AHR_EDEVICE, "unexpected exception");
    }
}

void ahr_wl_destroy(ahr_wl* h) {
    if (!h) return;
    try {
        delete reinterpret_cast<ahr::WlIndex*>(h);
    } catch (...) {
    }
    ahr::flush_frees();
}

}  // extern "C"
