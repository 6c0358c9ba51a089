// Half-perimeter wirelength of every placement in a signal: per net and per
// (x, y) column pair, (max - min) of the pin x plus that of the pin y, pin
// position = instance position + pin offset, in float64.
//
// A workgroup takes kBT nets at a time.  Their pins are consecutive, so they
// are read in windows of kWindow pins with one lane a pin (coalesced node and
// offset loads, every lane's position gathers in flight together) and left in
// LDS; then one thread a net runs over its pins there.  Nets with more than
// a wave's worth of pins are left out of the windows and summed by the whole
// workgroup, in net order.  Workgroup totals go to a partial-sum buffer,
// which one workgroup adds in a fixed order, so the result is deterministic
// and no list of the big nets is needed: the pass reads the netlist arrays
// alone.
//
// What bounds it: the position gathers, a line each from a table that only
// the Infinity Cache holds (about 18 ps a pin; 26 of the 84 us of a 1.1M-cell
// netlist without big nets).  8 lanes a net, which ran a chain of three
// dependent loads with most lanes idle (60 % of the nets have 2 pins), and
// one workgroup after another over the big nets took 61 us at 210k cells and
// 4 columns (35 now), 158 at 1.1M (134).  A net's thread reads a pin's pair in
// one 16-byte read: in arrays an axis, calls with 8 columns took 41 us at 2,000
// and 20,000 cells (29 now, 34 with the 8 lanes) and 275 at 2.2M (211, 373).
//
// ahr_hpwl draws the partial-sum buffer from the library's stream-ordered
// pool for each call, so calls on different streams share no memory.
#include "ahr_internal.hpp"
#include "device_util.hpp"

namespace ahr {

namespace {

constexpr int kBT = 256;
constexpr int kMaxGrid = 8192;      // workgroups, each of a multiple of kBT nets
constexpr int kMaxPairs = 4;        // ncols <= 8
constexpr size_t kPartialElems = static_cast<size_t>(kMaxGrid) * kMaxPairs;

// Pins a window holds: 16 P bytes of LDS each, four workgroups a CU or more.
template <int P>
constexpr int kWindow = P <= 2 ? 1024 : 512;

// Big nets up to this many pins take one wave, longer ones the workgroup, as
// does a batch's only big net.  At 7,000 and 210,000 cells (53 and 1,025 big
// nets) and 4 columns a call takes 23 and 41 us; with up to four big nets of a
// batch by the workgroup, one after another, 27 and 43; with all of them 28 and
// 48; waves up to 512 pins 23 and 44, up to 8,192 23 and 41.  A batch's only
// one by a wave is as fast (2,000 to 2.2M cells within 1 %).
constexpr int kWaveNet = 2048;
constexpr int kFewBig = 1;

template <int P>
__device__ __forceinline__ void bounds_init(double* lo, double* hi) {
#pragma unroll
    for (int c = 0; c < 2 * P; ++c) {
        lo[c] = 1e300;
        hi[c] = -1e300;
    }
}

// (a NaN coordinate moves no bound)
__device__ __forceinline__ void bound(double x, double& lo, double& hi) {
    lo = __builtin_fmin(lo, x);
    hi = __builtin_fmax(hi, x);
}

// Bounds over pins [p0, p1) of one net by W waves (t: the lane among them).
template <int P, int W>
__device__ __forceinline__ void net_bounds(const float* __restrict__ pos, const int32_t* __restrict__ pin_node,
                                           const float* __restrict__ pin_off, int p0, int p1, int t, double* lo,
                                           double* hi) {
    constexpr int U = P <= 2 ? 4 : 2;        // pins in flight a lane (a repeated last pin changes no bound)
    bounds_init<P>(lo, hi);
    for (int q = p0 + t; q < p1; q += U * W * kWave) {
        int v[U];
        float off[U][2], g[U][2 * P];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = q + u * W * kWave < p1 ? q + u * W * kWave : p1 - 1;
            v[u] = pin_node[p];
            off[u][0] = pin_off[2 * p];
            off[u][1] = pin_off[2 * p + 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 2 * P; ++c) g[u][c] = pos[static_cast<int64_t>(v[u]) * (2 * P) + c];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 2 * P; ++c)
                bound(static_cast<double>(g[u][c]) + static_cast<double>(off[u][c & 1]), lo[c], hi[c]);
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 2 * P; ++c) {
            lo[c] = __builtin_fmin(lo[c], __shfl_xor(lo[c], o));
            hi[c] = __builtin_fmax(hi[c], __shfl_xor(hi[c], o));
        }
}

template <int P>
__global__ void __launch_bounds__(kBT, 4) k_hpwl(const float* __restrict__ pos, const int32_t* __restrict__ net_ptr,
                                              int32_t n_nets, int32_t per, const int32_t* __restrict__ pin_node,
                                              const float* __restrict__ pin_off, double* __restrict__ partial) {
    constexpr int T = kWindow<P>, U = T / kBT;
    __shared__ double2 win[P][T];
    __shared__ double ext[2 * P][2][kBT / kWave];
    __shared__ double red[kBT / kWave];
    __shared__ int cnt[kBT / kWave];
    __shared__ int bstart[kBT], blen[kBT];      // the batch's big nets, in net order
    const int64_t lo_net = static_cast<int64_t>(blockIdx.x) * per;
    const int64_t hi_net = lo_net + per < n_nets ? lo_net + per : n_nets;
    double tot[P];
#pragma unroll
    for (int c = 0; c < P; ++c) tot[c] = 0;
    double lo[2 * P], hi[2 * P];
    auto add = [&]() {
#pragma unroll
        for (int c = 0; c < P; ++c) tot[c] += (hi[2 * c] - lo[2 * c]) + (hi[2 * c + 1] - lo[2 * c + 1]);
    };

    for (int64_t c0 = lo_net; c0 < hi_net; c0 += kBT) {
        const int64_t e = c0 + threadIdx.x;
        const int64_t last = c0 + kBT < hi_net ? c0 + kBT : hi_net;
        const int first = net_ptr[c0];
        const int p0 = net_ptr[e < last ? e : last], p1 = net_ptr[e < last ? e + 1 : last];
        const bool big = p1 - p0 > kWave;
        int nb;
        const int k = block_rank<kBT>(big, cnt, &nb);
        if (big) {
            bstart[k] = p0;
            blen[k] = p1 - p0;
        }
        __syncthreads();
        // the batch's pins without the big nets' are counted from 0; pins
        // of big nets before place q of that count: shift(q)
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
        bounds_init<P>(lo, hi);
        for (int at = 0; at < n; at += T) {
            int v[U];
            float ox[U], oy[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = at + static_cast<int>(threadIdx.x) + u * kBT, qc = q < n ? q : n - 1;
                const int p = first + qc + shift(qc);
                v[u] = pin_node[p];
                ox[u] = pin_off[2 * p];
                oy[u] = pin_off[2 * p + 1];
            }
            float g[U][2 * P];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < 2 * P; ++c) g[u][c] = pos[static_cast<int64_t>(v[u]) * (2 * P) + c];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < P; ++c)
                    win[c][threadIdx.x + u * kBT] =
                        make_double2(static_cast<double>(g[u][2 * c]) + static_cast<double>(ox[u]),
                                     static_cast<double>(g[u][2 * c + 1]) + static_cast<double>(oy[u]));
            __syncthreads();
            const int a = q0 > at ? q0 - at : 0, b = q1 < at + T ? q1 - at : T;
            constexpr int R = 4;
            for (int i = a; i < b; i += R) {         // R pins' reads at once (the last one repeats)
                double2 x[R][P];
#pragma unroll
                for (int u = 0; u < R; ++u)
#pragma unroll
                    for (int c = 0; c < P; ++c) x[u][c] = win[c][i + u < b ? i + u : b - 1];
#pragma unroll
                for (int u = 0; u < R; ++u)
#pragma unroll
                    for (int c = 0; c < P; ++c) {
                        bound(x[u][c].x, lo[2 * c], hi[2 * c]);
                        bound(x[u][c].y, lo[2 * c + 1], hi[2 * c + 1]);
                    }
            }
            __syncthreads();
        }
        if (q1 > q0) add();
        // the big nets: a wave each, the longest by the workgroup
        const int wave_net = nb > kFewBig ? kWaveNet : 0;
        for (int b = wave_id(); b < nb; b += kBT / kWave) {
            if (blen[b] > wave_net) continue;
            net_bounds<P, 1>(pos, pin_node, pin_off, bstart[b], bstart[b] + blen[b], lane_id(), lo, hi);
            if (lane_id() == 0) add();
        }
        for (int b = 0; b < nb; ++b) {
            if (blen[b] <= wave_net) continue;       // (the same in every thread)
            net_bounds<P, kBT / kWave>(pos, pin_node, pin_off, bstart[b], bstart[b] + blen[b], threadIdx.x, lo, hi);
            __syncthreads();
            if (lane_id() == 0) {
#pragma unroll
                for (int c = 0; c < 2 * P; ++c) {
                    ext[c][0][wave_id()] = lo[c];
                    ext[c][1][wave_id()] = hi[c];
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                for (int w = 1; w < kBT / kWave; ++w)
#pragma unroll
                    for (int c = 0; c < 2 * P; ++c) {
                        lo[c] = ext[c][0][w] < lo[c] ? ext[c][0][w] : lo[c];
                        hi[c] = ext[c][1][w] > hi[c] ? ext[c][1][w] : hi[c];
                    }
                add();
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < P; ++c) {
        double s = block_sum_f64<kBT>(tot[c], red);
        if (threadIdx.x == 0) partial[static_cast<int64_t>(blockIdx.x) * kMaxPairs + c] = s;
    }
}

// The workgroup partials in a fixed order: thread t adds partials t,
// t + kFinalBT, ... (all loaded at once), then a fixed block reduction.
constexpr int kFinalBT = 1024;
constexpr int kFinalPer = (kMaxGrid + kFinalBT - 1) / kFinalBT;

__global__ void __launch_bounds__(kFinalBT) k_hpwl_final(const double* __restrict__ partial, int nparts, int npairs,
                                                         double* __restrict__ out) {
    __shared__ double red[kFinalBT / kWave];
    for (int c = 0; c < npairs; ++c) {
        double v[kFinalPer];
#pragma unroll
        for (int u = 0; u < kFinalPer; ++u) {
            const int b = static_cast<int>(threadIdx.x) + u * kFinalBT;
            v[u] = partial[(b < nparts ? b : nparts - 1) * kMaxPairs + c];
        }
        double s = 0;
#pragma unroll
        for (int u = 0; u < kFinalPer; ++u) s += static_cast<int>(threadIdx.x) + u * kFinalBT < nparts ? v[u] : 0.0;
        s = block_sum_f64<kFinalBT>(s, red);
        if (threadIdx.x == 0) out[c] = s;
    }
}

// Nets per workgroup: kBT, or the multiple that stays within kMaxGrid.
int32_t hpwl_per(int32_t n_nets) {
    const int64_t batches = (static_cast<int64_t>(n_nets) + kBT - 1) / kBT;
    return static_cast<int32_t>((batches + kMaxGrid - 1) / kMaxGrid) * kBT;
}

int hpwl_grid(int32_t n_nets) {
    return n_nets < 1 ? 1 : static_cast<int>(grid_for(n_nets, hpwl_per(n_nets)));
}

template <int P>
void hpwl_p(const ahr_netlist& nl, const float* pos, double* out, double* partial, hipStream_t s) {
    const int grid = hpwl_grid(nl.n_nets);
    hipLaunchKernelGGL(k_hpwl<P>, dim3(grid), dim3(kBT), 0, s, pos, nl.net_ptr, nl.n_nets, hpwl_per(nl.n_nets),
                       nl.pin_node, nl.pin_off, partial);
    AHR_LAUNCHED("k_hpwl");
    hipLaunchKernelGGL(k_hpwl_final, dim3(1), dim3(kFinalBT), 0, s, partial, grid, P, out);
    AHR_LAUNCHED("k_hpwl_final");
}

}  // namespace

void hpwl_launch(const ahr_netlist& nl, const float* pos, int32_t ncols, double* out, double* partial,
                 hipStream_t s) {
    switch (ncols) {
        case 2: hpwl_p<1>(nl, pos, out, partial, s); break;
        case 4: hpwl_p<2>(nl, pos, out, partial, s); break;
        case 8: hpwl_p<4>(nl, pos, out, partial, s); break;
        default: throw Error{AHR_EUNSUPPORTED, "hpwl needs ncols of 2, 4 or 8"};
    }
}

size_t hpwl_partial_elems() { return kPartialElems; }

void run_hpwl(const ahr_netlist& nl, const float* pos, int32_t ncols, double* out, hipStream_t s) {
    ProfScope ps(kStageHpwl, s);
    DevBuf<double> partial;
    partial.ensure(static_cast<size_t>(hpwl_grid(nl.n_nets)) * kMaxPairs, s);
    hpwl_launch(nl, pos, ncols, out, partial.p, s);
    partial.release(s);
}

}  // namespace ahr
