// Learned surrogate of the refinement filter (a project addition; the
// paper has no learned component).  For every (instance row, column):
//   h_j = (T^j X) for j = 0..3 (h_0 = X), m_c / s_c = mean / std of h_3 over
//   movable rows, r_c = root mean square of h_0 - h_3 over movable rows,
//   f = [(h0 - h3)/r_c, (h1 - h3)/r_c, (h2 - h3)/r_c, (h3 - m_c)/s_c,
//        log1p(d), hsum/d, log(s_c / r_c)],
//   o = w3 . relu(W2 relu(W1 f + b1) + b2) + b3,
//   y = beta_0 h0 + beta_1 h1 + beta_2 h2 + beta_3 h3 + r_c o   (fixed rows keep their input).
// r_c, the displacement of three hops, is a length of the graph's local
// neighbourhoods while s_c grows with the die, so the scaled differences and
// the output correction keep their size on netlists of any size.
//
// Inference runs the three layers on the matrix cores: 16 samples per
// wavefront, bfloat16 operands, float32 accumulation.  Every layer is
// computed transposed (hidden x samples): the accumulator of one 16-row
// output tile leaves lane l with rows 4(l/16)..4(l/16)+3 of sample l%16.
// Every layer uses gfx950's v_mfma_f32_16x16x32_bf16, whose B operand gives
// lane l eight K slots 8(l/16)..8(l/16)+7.  In layer 1 the 7 features, padded
// to 8, are one lane group's slots and the others' are zeros (mlp_tile).
// Layers 2 and 3 contract over the 64 hidden units: the lane's rows of two
// output tiles fill its slots (slots 8g..8g+3 hold hidden units 32p+4g..+3,
// slots 8g+4..8g+7 hold 32p+16+4g..+3), and the weights are loaded into the A
// operand with the same permutation of K, so no data moves between lanes.
//
// Training runs forward and backward with the same bfloat16 rounding points
// (weights, features and hidden activations) and float32 accumulation,
// gradients straight through the rounding, accumulated per workgroup in a
// fixed order and reduced in a fixed order.
#include <algorithm>

#include "ahr_internal.hpp"
#include "device_util.hpp"

namespace ahr {

namespace {

constexpr int kBT = 256;
constexpr int kH = AHR_MLP_HIDDEN;      // 64
constexpr int kFP = 8;                  // padded feature count
constexpr int kNP = AHR_MLP_NPARAM;     // 4801
constexpr int oW1 = 0, oB1 = kH * kFP, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH, oB3 = oW3 + kH;
static_assert(oB3 + 1 == kNP, "parameter layout");

typedef short v2s __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

// Hidden unit of K slot q (0..31) of chunk p in the layers contracting over
// the hidden units (see above).
__device__ __forceinline__ int hid(int p, int q) { return 32 * p + ((q & 4) ? 16 : 0) + 4 * (q >> 3) + (q & 3); }

__device__ __forceinline__ v4f mfma32(v8s a, v8s b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0,
                                                  0);
}

// float32 -> bfloat16, round to nearest even (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ short bf16_bits(float x) { return __builtin_bit_cast(short, static_cast<__bf16>(x)); }
__device__ __forceinline__ float bf16_value(short b) { return static_cast<float>(__builtin_bit_cast(__bf16, b)); }
__device__ __forceinline__ float bf16_round(float x) { return static_cast<float>(static_cast<__bf16>(x)); }

// ---------------------------------------------------------------- inference

// relu then bfloat16 of two values, as relu of the bfloat16 values (rounding
// keeps the sign): one packed conversion, then one packed signed 16-bit max
// with 0, since a negative bfloat16 has its sign bit set.
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v2s relu_bf16x2(float a, float b) {
    const v2bf t = __builtin_convertvector((v2f{a, b}), v2bf);
    return __builtin_elementwise_max(__builtin_bit_cast(v2s, t), v2s{0, 0});
}

__device__ __forceinline__ v4s relu_bf16x4(v4f acc) {
    const v2s lo = relu_bf16x2(acc[0], acc[1]), hi = relu_bf16x2(acc[2], acc[3]);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
}

struct MlpRegs {
    v8s w1[4];        // A tiles of W1 (hidden 16m..), features 0..7 in the K slots of every lane group
    v8s w2[8];        // A tiles of W2 (out 16n.., in chunk p of 32, K permuted), index 2n + p
    v8s w3[2];        // A tiles with w3 in every row (chunk p, K permuted)
    float b1[16], b2[16];
    float b3;
    bool wild;        // W1 has a bfloat16 infinity or NaN (the same in every lane)
};

// OneGroup: the samples' features always lie in lanes 0..15 (see mlp_tile).
template <bool OneGroup>
__device__ __forceinline__ void load_mlp(const float* __restrict__ P, MlpRegs& R) {
    const int l = lane_id(), i = l & 15, g = l >> 4;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int k = 4 * g + j;
            R.b1[4 * m + j] = P[oB1 + 16 * m + k];
            R.b2[4 * m + j] = P[oB2 + 16 * m + k];
        }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int k = 0; k < kFP; ++k) R.w1[m][k] = bf16_bits(P[oW1 + (16 * m + i) * kFP + k]);
    bool wild = false;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int k = 0; k < kFP; ++k) wild |= (R.w1[m][k] & 0x7f80) == 0x7f80;
    R.wild = __any(wild);
    if (OneGroup && g != 0)
#pragma unroll
        for (int m = 0; m < 4; ++m) R.w1[m] = v8s{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int h = hid(p, 8 * g + j);
            R.w3[p][j] = bf16_bits(P[oW3 + h]);
#pragma unroll
            for (int n = 0; n < 4; ++n) R.w2[2 * n + p][j] = bf16_bits(P[oW2 + (16 * n + i) * kH + h]);
        }
    R.b3 = P[oB3];
}

// A sample's eight features as one lane's B operand.
__device__ __forceinline__ v4i pack_features(const float F[kFP]) {
    v4i x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const v2bf t = __builtin_convertvector((v2f{F[2 * k], F[2 * k + 1]}), v2bf);
        x[k] = __builtin_bit_cast(int, t);
    }
    return x;
}

// One tile of 16 samples: x holds the features of sample l%16 in one group of
// 16 lanes and zeros in the other three, whose K slots so add nothing; the
// result of sample l%16 is in every lane.  Wild: with weights that are not
// finite, where 0 x inf would be NaN, which the relu may turn into 0; the
// weights beside the zeros are zeroed as well (own: the features' group).
template <bool Wild>
__device__ __forceinline__ float mlp_tile(const MlpRegs& R, v4i x, int own) {
    v4s a1[4], a2[4];
    // each layer's accumulator starts at its bias (float32)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        v4f acc = {R.b1[4 * m], R.b1[4 * m + 1], R.b1[4 * m + 2], R.b1[4 * m + 3]};
        v8s w = R.w1[m];
        if (Wild && lane_id() >> 4 != own) w = v8s{0, 0, 0, 0, 0, 0, 0, 0};
        acc = mfma32(w, __builtin_bit_cast(v8s, x), acc);
        a1[m] = relu_bf16x4(acc);
    }
    // the lane's rows of output tiles 2p and 2p+1: the B operand of chunk p
    v8s b1[2], b2[2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b1[p][j] = a1[2 * p][j];
            b1[p][4 + j] = a1[2 * p + 1][j];
        }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        v4f acc = {R.b2[4 * n], R.b2[4 * n + 1], R.b2[4 * n + 2], R.b2[4 * n + 3]};
#pragma unroll
        for (int p = 0; p < 2; ++p) acc = mfma32(R.w2[2 * n + p], b1[p], acc);
        a2[n] = relu_bf16x4(acc);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b2[p][j] = a2[2 * p][j];
            b2[p][4 + j] = a2[2 * p + 1][j];
        }
    v4f acc = {R.b3, R.b3, R.b3, R.b3};
#pragma unroll
    for (int p = 0; p < 2; ++p) acc = mfma32(R.w3[p], b2[p], acc);
    return acc[0];
}

// o[s] for a flat list of feature rows feats[n][8].
__global__ void __launch_bounds__(kBT) k_mlp_forward(const float* __restrict__ P, const float* __restrict__ feats,
                                                     int64_t n, float* __restrict__ o) {
    MlpRegs R;
    load_mlp<true>(P, R);
    const int l = lane_id(), g = l >> 4;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kBT / kWave);
    const int64_t ntiles = (n + 15) / 16;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (kBT / kWave) + wave_id(); t < ntiles; t += waves) {
        const int64_t smp = t * 16 + (l & 15);
        float F[kFP] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (smp < n && g == 0) {
            const float4 u = reinterpret_cast<const float4*>(feats + smp * kFP)[0];
            const float4 v = reinterpret_cast<const float4*>(feats + smp * kFP)[1];
            F[0] = u.x, F[1] = u.y, F[2] = u.z, F[3] = u.w;
            F[4] = v.x, F[5] = v.y, F[6] = v.z, F[7] = v.w;
        }
        float r = mlp_tile<false>(R, pack_features(F), 0);
        if (l < 16 && smp < n) o[smp] = r;
    }
}

// Signal value h of (execution row, column) from the scaled chain z
// (inv_s = 1 / s of the row; 0 for an isolated row, whose value is its input).
__device__ __forceinline__ float unscale(const float* z, int C, int r, int c, float inv_s, const float* in,
                                         const int32_t* perm) {
    return inv_s > 0.f ? z[static_cast<int64_t>(r) * C + c] * inv_s : in[static_cast<int64_t>(perm[r]) * C + c];
}

struct LearnArgs {
    const float* z0;        // the expanded input, scaled like the hops
    const float* z1;
    const float* z2;
    const float* z3;
    const float* scale;
    const double* deg;
    const float* hsum;
    const float* stats;     // [3][C]: mean and std of h3, rms of h0 - h3
    float4* rowf;           // [n_inst] per execution row: 1/s, log1p(d), hsum/d, row code (bits)
    const float* in;
    float* out;
    float* feats;           // optional [n_inst * C][8], instance order
    float* hops;            // optional [4][n_inst][C], instance order
    const uint8_t* flags;
    const int32_t* perm;
    const float* params;
    float beta[4];
    int32_t n_inst;
    int write_out;
};

// Per-row inputs of the features, once per row instead of once per column:
// 1/s, log1p(d), hsum/d (the last two in float64, then rounded), and the
// row's instance with its fixed flag in the sign bit (the bits of w), so the
// network's epilogue needs no dependent load to find where its result goes.
__device__ __forceinline__ int row_inst(int code) { return code & 0x7fffffff; }
__device__ __forceinline__ bool row_fixed(int code) { return code < 0; }

__device__ __forceinline__ float4 row_feat(float s, double d, float hs, int inst, uint8_t flags) {
    const int code = inst | ((flags & AHR_NODE_FIXED) ? static_cast<int>(0x80000000u) : 0);
    return make_float4(s > 0.f ? 1.f / s : 0.f, static_cast<float>(log1p(d)),
                       d > 0 ? static_cast<float>(static_cast<double>(hs) / d) : 0.f, __int_as_float(code));
}

// One sample's inputs: the scaled hops z_j (h = z_j / s once the row's 1/s
// is known) and the row inputs, none depending on another, so the next
// group's loads are in flight while the current one runs through the
// network.
struct SampleIn {
    float h[4];
    float4 rf;
};

template <int C>
__device__ __forceinline__ SampleIn sample_load(const LearnArgs& a, int64_t smp) {
    SampleIn t;
    const int64_t r = smp / C;
    t.h[0] = t.h[1] = t.h[2] = t.h[3] = 0.f;
    t.rf = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < a.n_inst) {
        t.rf = a.rowf[r];
        t.h[0] = a.z0[smp];
        t.h[1] = a.z1[smp];
        t.h[2] = a.z2[smp];
        t.h[3] = a.z3[smp];
    }
    return t;
}

// The hops' values from the loaded z: h = z / s, or the input for a row
// with s = 0 (isolated: every power of the operator keeps its value), which
// is rare, so its dependent load sits in a branch of its own.
template <int C>
__device__ __forceinline__ void sample_unscale(const LearnArgs& a, SampleIn& t, int64_t smp) {
    const float inv_s = t.rf.x;
    if (inv_s > 0.f) {
#pragma unroll
        for (int j = 0; j < 4; ++j) t.h[j] *= inv_s;
    } else if (smp / C < a.n_inst) {
        const float v = a.in[static_cast<int64_t>(row_inst(__float_as_int(t.rf.w))) * C + smp % C];
#pragma unroll
        for (int j = 0; j < 4; ++j) t.h[j] = v;
    }
}

// The learned filter over the instance rows, 64 samples (64/C rows x C
// columns) per wavefront and step: each lane loads and featurises its own
// sample (its column is the same at every step, as 64 % C == 0, so its
// column statistics are loaded once), then the network runs the four
// 16-sample matrix-core tiles in turn, each fed by the lanes that own its
// samples (the other lanes' K slots hold zeros), which find their results in
// place and write them.  The next step's loads are in flight meanwhile.  A
// sample's result does not depend on its tile's other samples.
// What bounds it: the matrix and conversion steps of a tile follow one another
// (14 products, 32 conversions), with three waves a SIMD to fill in.  880k
// cells x 4 columns: 60 us, against 84 with the features and results moved by
// nine shuffles a tile.
template <int C>
__global__ void __launch_bounds__(kBT) k_mlp_learned(LearnArgs a) {
    MlpRegs R;
    load_mlp<false>(a.params, R);
    const int l = lane_id(), g = l >> 4;
    const int c = l % C;
    const float mc = a.stats[c], sc = a.stats[C + c], rc = a.stats[2 * C + c];
    const float inv_sc = 1.f / sc, inv_rc = 1.f / rc;
    const float lsr = static_cast<float>(log(static_cast<double>(sc) / static_cast<double>(rc)));
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kBT / kWave);
    const int64_t nsteps = (static_cast<int64_t>(a.n_inst) * C + kWave - 1) / kWave;
    int64_t t = static_cast<int64_t>(blockIdx.x) * (kBT / kWave) + wave_id();
    SampleIn cur = sample_load<C>(a, t * kWave + l);
    for (; t < nsteps; t += waves) {
        const SampleIn nxt = sample_load<C>(a, (t + waves) * kWave + l);
        const int64_t smp = t * kWave + l;
        sample_unscale<C>(a, cur, smp);
        float F[8];
        F[0] = (cur.h[0] - cur.h[3]) * inv_rc;
        F[1] = (cur.h[1] - cur.h[3]) * inv_rc;
        F[2] = (cur.h[2] - cur.h[3]) * inv_rc;
        F[3] = (cur.h[3] - mc) * inv_sc;
        F[4] = cur.rf.y;
        F[5] = cur.rf.z;
        F[6] = lsr;
        F[7] = 0.f;
        const v4i x = pack_features(F);
        float mine = 0.f;
#pragma unroll 2
        for (int j = 0; j < kWave / 16; ++j) {
            v4i own;
#pragma unroll
            for (int k = 0; k < 4; ++k) own[k] = g == j ? x[k] : 0;
            const float o = R.wild ? mlp_tile<true>(R, own, j) : mlp_tile<false>(R, own, j);     // of sample 16 j + i
            if (g == j) mine = o;
        }
        const int64_t r = smp / C;
        if (r < a.n_inst) {
            const int code = __float_as_int(cur.rf.w), inst = row_inst(code);
            const int64_t oc = static_cast<int64_t>(inst) * C + c;
            if (a.feats) {
                float* fp = a.feats + oc * kFP;
                fp[0] = F[0], fp[1] = F[1], fp[2] = F[2], fp[3] = F[3];
            }
            if (a.hops) {
                const int64_t nc = static_cast<int64_t>(a.n_inst) * C;
#pragma unroll
                for (int j = 0; j < 4; ++j) a.hops[j * nc + oc] = cur.h[j];
            }
            if (a.write_out) {
                float y = a.beta[0] * cur.h[0] + a.beta[1] * cur.h[1] + a.beta[2] * cur.h[2] + a.beta[3] * cur.h[3] +
                          rc * mine;
                a.out[oc] = row_fixed(code) ? a.in[oc] : y;
            }
        }
        cur = nxt;
    }
}

// Features 4..7 of every sample (the row values, the column's log(s/r) and
// the padding), for the exported feature rows.
template <int C>
__global__ void k_feature_row(LearnArgs a) {
    int64_t smp = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (smp >= static_cast<int64_t>(a.n_inst) * C) return;
    const int r = static_cast<int>(smp / C), c = static_cast<int>(smp % C);
    const float4 rf = a.rowf[r];
    const double lsr = log(static_cast<double>(a.stats[C + c]) / static_cast<double>(a.stats[2 * C + c]));
    *reinterpret_cast<float4*>(a.feats + (static_cast<int64_t>(a.perm[r]) * C + c) * kFP + 4) =
        make_float4(rf.y, rf.z, static_cast<float>(lsr), 0.f);
}

// Column statistics over movable instance rows in one pass (fixed grid,
// float64 partials added in a fixed order): per column the sums of h3 - c
// and (h3 - c)^2, with c the column's value at execution row 0 (a shift that
// lies inside the data, so the variance E[(h3-c)^2] - E[h3-c]^2 loses few
// digits), and of (h0 - h3)^2.
constexpr int kStatGrid = 512;

// One row's C values of a scaled hop.
template <int C>
struct alignas(C * sizeof(float) < 16 ? C * sizeof(float) : 16) ZRow {
    float v[C];
};

// The same pass forms the rows' inputs of the features (rowf).  The loads of
// kStatRows rows a thread are in flight together: 880k cells x 4 columns take
// 22 us, against 13 us for a kernel of rowf alone and 23 us for the sums with
// a row's loads one after another.
constexpr int kStatRows = 4;

template <int C>
__global__ void __launch_bounds__(kBT) k_colstat(LearnArgs a, double* __restrict__ part) {
    constexpr int W = 3 * C + 1;
    __shared__ double red[W][kBT / kWave];
    double shift[C];
#pragma unroll
    for (int c = 0; c < C; ++c) shift[c] = 0;
    if (a.n_inst > 0) {
        const float inv_s0 = a.scale[0] > 0.f ? 1.f / a.scale[0] : 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c) shift[c] = unscale(a.z3, C, 0, c, inv_s0, a.in, a.perm);
    }
    double acc[W];
#pragma unroll
    for (int c = 0; c < W; ++c) acc[c] = 0;
    constexpr int64_t kStep = static_cast<int64_t>(kStatGrid) * kBT;
    for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * kBT + threadIdx.x; r0 < a.n_inst; r0 += kStatRows * kStep) {
        float s[kStatRows], hs[kStatRows];
        double deg[kStatRows];
        int inst[kStatRows];
        uint8_t fl[kStatRows];
        ZRow<C> z3[kStatRows], z0[kStatRows];
#pragma unroll
        for (int u = 0; u < kStatRows; ++u) {
            const int64_t r = r0 + u * kStep < a.n_inst ? r0 + u * kStep : r0;
            inst[u] = a.perm[r];
            s[u] = a.scale[r];
            hs[u] = a.hsum[r];
            deg[u] = a.deg[r];
            z3[u] = reinterpret_cast<const ZRow<C>*>(a.z3)[r];
            z0[u] = reinterpret_cast<const ZRow<C>*>(a.z0)[r];
        }
#pragma unroll
        for (int u = 0; u < kStatRows; ++u) fl[u] = a.flags[inst[u]];
#pragma unroll
        for (int u = 0; u < kStatRows; ++u) {
            const int64_t r = r0 + u * kStep;
            if (r >= a.n_inst) break;
            const float4 rf = row_feat(s[u], deg[u], hs[u], inst[u], fl[u]);
            a.rowf[r] = rf;
            const int code = __float_as_int(rf.w);
            if (row_fixed(code)) continue;
            const float inv_s = rf.x;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                float h3 = z3[u].v[c] * inv_s, h0 = z0[u].v[c] * inv_s;
                if (!(inv_s > 0.f)) h3 = h0 = a.in[static_cast<int64_t>(row_inst(code)) * C + c];     // isolated
                const double h = h3, d = h - shift[c], d0 = h0 - h;
                acc[c] += d;
                acc[C + c] += d * d;
                acc[2 * C + c] += d0 * d0;
            }
            acc[3 * C] += 1.0;
        }
    }
    block_sums_f64<kBT>(acc, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < W; ++c) part[static_cast<int64_t>(blockIdx.x) * W + c] = acc[c];
    }
}

// stats [3][C]: mean and standard deviation of h3, rms of h0 - h3 (a zero
// deviation or rms becomes 1).  One workgroup: each thread adds a fixed
// stride of the partials in order, then a fixed block reduction.
template <int C>
__global__ void __launch_bounds__(kBT) k_colstat_final(LearnArgs a, const double* __restrict__ part,
                                                       float* __restrict__ stats) {
    constexpr int W = 3 * C + 1;
    __shared__ double red[W][kBT / kWave];
    double tot[W];
#pragma unroll
    for (int c = 0; c < W; ++c) tot[c] = 0;
    for (int b = threadIdx.x; b < kStatGrid; b += kBT)
#pragma unroll
        for (int c = 0; c < W; ++c) tot[c] += part[static_cast<int64_t>(b) * W + c];
    block_sums_f64<kBT>(tot, red);
    if (threadIdx.x != 0) return;
    const double n = tot[3 * C];
    const float inv_s0 = a.n_inst > 0 ? a.rowf[0].x : 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double shift = a.n_inst > 0 ? unscale(a.z3, C, 0, c, inv_s0, a.in, a.perm) : 0.0;
        const double m1 = n > 0 ? tot[c] / n : 0.0;
        const double var = n > 0 ? tot[C + c] / n - m1 * m1 : 0.0;
        const double sd = var > 0 ? sqrt(var) : 0.0;
        const double rms = n > 0 ? sqrt(tot[2 * C + c] / n) : 0.0;
        stats[c] = n > 0 ? static_cast<float>(shift + m1) : 0.f;
        stats[C + c] = sd > 0 ? static_cast<float>(sd) : 1.f;
        stats[2 * C + c] = rms > 0 ? static_cast<float>(rms) : 1.f;
    }
}

// ---------------------------------------------------------------- training

constexpr int kTS = 32;           // samples per tile
constexpr int kGradGrid = 240;    // workgroups of the float32-operand form (fixed: fixes the summation order)
constexpr int kGradMax = 512;     // most workgroups of the matrix-core form: two per CU, its occupancy

// bfloat16 of relu(z), NaN -> 0: the median of z, 0 and infinity (inf: a
// register, since with a constant the compiler takes two instructions).  The
// empty asm keeps the packed words as they are: the compiler otherwise
// converts each half again for the masks taken from them.
__device__ __forceinline__ v4s relu_pack(v4f z, float inf) {
    auto relu = [&](float x) { return __builtin_amdgcn_fmed3f(x, 0.f, inf); };
    v2i w = {__builtin_bit_cast(int, __builtin_convertvector((v2f{relu(z[0]), relu(z[1])}), v2bf)),
             __builtin_bit_cast(int, __builtin_convertvector((v2f{relu(z[2]), relu(z[3])}), v2bf))};
    asm("" : "+v"(w));
    return __builtin_bit_cast(v4s, w);
}

__device__ __forceinline__ v8s join(v4s a, v4s b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

// All ones in the halves whose (non-negative) bfloat16 is not zero.
__device__ __forceinline__ v4i nonzero(v8s a) {
    const v4i w = __builtin_bit_cast(v4i, a);
    v4i m;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int x = w[k];
        m[k] = __builtin_bit_cast(int, v2s{0, 0} - __builtin_elementwise_min(__builtin_bit_cast(v2s, x), v2s{1, 1}));
    }
    return m;
}

__device__ __forceinline__ v8s masked(v4i m, v8s a) {
    v4i w = m & __builtin_bit_cast(v4i, a);
    asm("" : "+v"(w));      // (whole words: the compiler otherwise ands the halves)
    return __builtin_bit_cast(v8s, w);
}

// From here on a float32 rounds to an infinite bfloat16.
constexpr float kBf16Over = 0x1.ffp127f;

// x = hi + mid + lo, each bfloat16 (exact for finite x whose parts are normal).
// Below kBf16Over, or with Far for any x: a finite one past it has the largest
// bfloat16 as its first part, an infinity is its first part alone (the rest
// would be inf - inf).
template <bool Far>
__device__ __forceinline__ void split3(v2f x, v2s (&p)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v2f top = x;
        if constexpr (Far)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (fabsf(x[k]) >= kBf16Over && fabsf(x[k]) < INFINITY) top[k] = copysignf(0x1.fep127f, x[k]);
        const v2bf h = __builtin_convertvector(top, v2bf);
        p[c] = __builtin_bit_cast(v2s, h);
        v2f rest = x - __builtin_convertvector(h, v2f);
        if constexpr (Far)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (fabsf(x[k]) == INFINITY) rest[k] = 0.f;
        x = rest;
    }
}

// A wave's 32 samples on their way to LDS: feature floats l, l + 64, ... and
// (lanes below 32) one target; zeros past sample n.
struct GradTile {
    float x[4], t;
};

__device__ __forceinline__ void load_grad_tile(const float* __restrict__ feats, const float* __restrict__ target,
                                               int64_t s0, int64_t n, GradTile& T) {
    const int l = lane_id();
    const int64_t left = n - s0;                 // >= 1
    const int nf = left < kTS ? static_cast<int>(left) * kFP : kTS * kFP;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = l + kWave * q;
        T.x[q] = feats[s0 * kFP + (e < nf ? e : nf - 1)];
        if (e >= nf) T.x[q] = 0.f;
    }
    T.t = target[s0 + (l < left ? l % kTS : 0)];
}

// The gradient with the inference's bfloat16 rounding points, on the matrix
// cores.  A wave takes 32 samples at a time.  Every product below has
// operands that are bfloat16 exactly (or float32 on the float32 matrix
// instruction), so nothing is rounded that the float32 form keeps:
//   z1, z2, o      weights, features and hidden activations are bfloat16 by
//                  the rounding points; b1 rides in layer 1's unused K slots
//                  as its three bfloat16 parts (x = hi + mid + lo holds all
//                  24 bits of a float32).
//   dz1            = [z1 > 0] do u,  u = W2^T (w3 [z2 > 0]): w3 masked is bfloat16.
//   gW2[h][k]      = w3_h sum_s [z2 > 0] do_s a1_sk: do_s as its three
//                  bfloat16 parts, one product each; gb2 the same without a1,
//                  gw3 = sum_s do_s a2 likewise.
//   gW1, gb1       sum over samples of dz1 (float32) times the features and a
//                  column of ones, with v_mfma_f32_16x16x4_f32.
// Contractions over hidden units need a lane to hold hidden units of one
// sample, contractions over samples need samples of one hidden unit.  A tile
// product gives one or the other by the order of its operands (the same
// registers), so z1 and z2 are formed both ways and nothing moves between
// lanes.  The weights' operands sit in LDS in fragment order.
//
// What bounds it: the matrix instructions, about 1,450 SIMD cycles per 16
// samples (three quarters of them in gW2 and gW1), beside about as many
// cycles of vector work (masks, packing).  1.6M samples take 0.161 ms where
// the LDS tiles in float32 took 13.28 (5,000: 39 against 89 us with Adam);
// the gradient's error against 64 bits went from 7.5e-7 to 4.5e-7.
__global__ void __launch_bounds__(kBT, 2) k_mlp_grad_mfma(const float* __restrict__ P, const float* __restrict__ feats,
                                                          const float* __restrict__ target, int64_t n, float inv_n,
                                                          float* __restrict__ part, double* __restrict__ loss_part) {
    __shared__ v8s w2f[8][kWave];        // W2 rows as operands (output 16n+i, K slots over the inputs), index 2n + p
    __shared__ v8s w2tf[8][kWave];       // W2 columns (input 16n+i, K slots over the outputs)
    __shared__ __attribute__((aligned(16))) float b2s[kH];
    // each wave's samples: 8 features (bfloat16 values), a one, zeros; the
    // row stride keeps gW1's reads (lane group g at rows 4g) off each other's banks
    constexpr int kXS = 20;
    __shared__ __attribute__((aligned(16))) float xs[kBT / kWave][kTS][kXS], ts[kBT / kWave][kTS];
    __shared__ float sum[kNP];
    __shared__ float gb2[kBT / kWave][kH];       // of the samples whose do may not be finite
    __shared__ double lsum[kBT / kWave];
    const int t = threadIdx.x, l = lane_id(), i = l & 15, g = l >> 4;
    (&gb2[0][0])[t] = 0.f;
    static_assert(kBT == kBT / kWave * kH, "one value a thread");
    for (int e = t; e < 8 * kWave; e += kBT) {
        const int q = e / kWave, el = e % kWave, ei = el & 15, eg = el >> 4, row = 16 * (q >> 1) + ei;
        v8s a, b;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int h = hid(q & 1, 8 * eg + j);
            a[j] = bf16_bits(P[oW2 + row * kH + h]);
            b[j] = bf16_bits(P[oW2 + h * kH + row]);
        }
        w2f[q][el] = a;
        w2tf[q][el] = b;
    }
    if (t < kH) b2s[t] = P[oB2 + t];
    for (int e = t; e < kNP; e += kBT) sum[e] = 0.f;
    for (int e = t; e < kBT / kWave * kTS * kXS; e += kBT)
        (&xs[0][0][0])[e] = e % kXS == kFP ? 1.f : 0.f;
    float inf = INFINITY;
    asm("" : "+s"(inf));
    // K slots of layer 1: the 8 features, then b1's three parts against ones
    v4s w1[4];
    v8s w3[2];
    float b2n[4];
    const float b3 = P[oB3];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        v2s bp[3];
        split3<true>(v2f{P[oB1 + 16 * m + i], 0.f}, bp);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const short wv = bf16_bits(P[oW1 + (16 * m + i) * kFP + 4 * (g & 1) + j]);
            w1[m][j] = g < 2 ? wv : g == 2 && j < 3 ? bp[j < 3 ? j : 0][0] : static_cast<short>(0);
        }
        b2n[m] = P[oB2 + 16 * m + i];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) w3[p][j] = bf16_bits(P[oW3 + hid(p, 8 * g + j)]);
    const short kOne = 0x3F80;           // bfloat16 1.0
    const v4s ones = {g == 2 ? kOne : short(0), g == 2 ? kOne : short(0), g == 2 ? kOne : short(0), 0};
    const v4f zero = {0.f, 0.f, 0.f, 0.f};
    v4f gw2[4][4], gw1[4], gv[4];        // gv: columns 0..2 gw3, 4..6 gb2 (one per part of do)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        gw1[m] = gv[m] = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) gw2[m][k] = zero;
    }
    float gb3 = 0.f;
    double loss = 0;
    // The loss of any one sample whose do may round to an infinite bfloat16 (an
    // infinity or NaN keeps it there for good): asked once a pair, where a test
    // of the eight do's took 4 % of the kernel.
    const double far_e = 0.99 * kBf16Over / (2.0 * inv_n), far_loss = far_e * far_e;
    __syncthreads();
    const int64_t npairs = (n + kTS - 1) / kTS;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kBT / kWave);
    int64_t pair = static_cast<int64_t>(blockIdx.x) * (kBT / kWave) + wave_id();
    GradTile cur;
    if (pair < npairs) load_grad_tile(feats, target, pair * kTS, n, cur);
    float (*X)[kXS] = xs[wave_id()];
    float* T = ts[wave_id()];
    for (; pair < npairs; pair += waves) {
#pragma unroll
        for (int q = 0; q < 4; ++q) X[(l + kWave * q) / kFP][l % kFP] = bf16_round(cur.x[q]);
        if (l < kTS) T[l] = cur.t;
        // (LDS serves a wave's accesses in order; the compiler keeps them so)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int left = n - pair * kTS < kTS ? static_cast<int>(n - pair * kTS) : kTS;
        if (pair + waves < npairs) load_grad_tile(feats, target, (pair + waves) * kTS, n, cur);
        v4s a1n[2][4], a2n[2][4];        // samples 4g..4g+3 of hidden unit 16m+i
        v4s dp[2][3];                    // the parts of do of samples 4g..4g+3
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const v4f xt = *reinterpret_cast<const v4f*>(&X[16 * u + i][4 * (g & 1)]);
            const v2bf x01 = __builtin_convertvector((v2f{xt[0], xt[1]}), v2bf);
            const v2bf x23 = __builtin_convertvector((v2f{xt[2], xt[3]}), v2bf);
            v4s x = __builtin_shufflevector(__builtin_bit_cast(v2s, x01), __builtin_bit_cast(v2s, x23), 0, 1, 2, 3);
            x = g < 2 ? x : ones;
            v4s h1[4], h2[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                h1[m] = relu_pack(__builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1[m], x, zero, 0, 0, 0), inf);
            const v8s a1t[2] = {join(h1[0], h1[1]), join(h1[2], h1[3])};
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const v8s wa = w2f[2 * m][l], wb = w2f[2 * m + 1][l];
                v4f zt = *reinterpret_cast<const v4f*>(&b2s[16 * m + 4 * g]);
                v4f zn = {b2n[m], b2n[m], b2n[m], b2n[m]};
                zt = mfma32(wa, a1t[0], zt);
                zn = mfma32(a1t[0], wa, zn);
                zt = mfma32(wb, a1t[1], zt);
                zn = mfma32(a1t[1], wb, zn);
                h2[m] = relu_pack(zt, inf);
                a2n[u][m] = relu_pack(zn, inf);
            }
            const v8s a2t[2] = {join(h2[0], h2[1]), join(h2[2], h2[3])};
            __builtin_amdgcn_sched_barrier(0);
            // o of samples 4g..4g+3, the same in every column
            v4f o = {b3, b3, b3, b3};
            o = mfma32(a2t[0], w3[0], o);
            o = mfma32(a2t[1], w3[1], o);
            const v4f want = *reinterpret_cast<const v4f*>(&T[16 * u + 4 * g]);
            v4f dO;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float e = 16 * u + 4 * g + j < left ? o[j] - want[j] : 0.f;
                dO[j] = 2.f * e * inv_n;
                loss += static_cast<double>(e) * e;
                gb3 += dO[j];
            }
            v2s p01[3], p23[3];
            *reinterpret_cast<v4f*>(&T[16 * u + 4 * g]) = dO;       // (for the far case below)
            split3<false>(v2f{dO[0], dO[1]}, p01);
            split3<false>(v2f{dO[2], dO[3]}, p23);
#pragma unroll
            for (int c = 0; c < 3; ++c) dp[u][c] = __builtin_shufflevector(p01[c], p23[c], 0, 1, 2, 3);
            // dz1 = [z1 > 0] do u, then gW1 and gb1
            const v8s q0 = masked(nonzero(a2t[0]), w3[0]), q1 = masked(nonzero(a2t[1]), w3[1]);
            float xb[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) xb[j] = X[16 * u + 4 * g + j][i];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                v4f uz = mfma32(q0, w2tf[2 * m][l], zero);
                uz = mfma32(q1, w2tf[2 * m + 1][l], uz);
                const v4f z1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, w1[m], zero, 0, 0, 0);
                a1n[u][m] = relu_pack(z1, inf);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float dz = z1[j] > 0.f ? dO[j] * uz[j] : 0.f;
                    gw1[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(dz, xb[j], gw1[m], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // contractions over the 32 samples: slots 8g..8g+3 hold tile 0's
        // samples 4g..4g+3, slots 8g+4..8g+7 tile 1's
        const bool far = __any(!(loss < far_loss));
        if (far) {      // split again, for any do; and gb2 here: 0 x inf in its product would be NaN for the dead units
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const v4f x = *reinterpret_cast<const v4f*>(&T[16 * u + 4 * g]);
                v2s p01[3], p23[3];
                split3<true>(v2f{x[0], x[1]}, p01);
                split3<true>(v2f{x[2], x[3]}, p23);
#pragma unroll
                for (int c = 0; c < 3; ++c) dp[u][c] = __builtin_shufflevector(p01[c], p23[c], 0, 1, 2, 3);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                float v = 0.f;
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float x = (bf16_value(dp[u][0][j]) + bf16_value(dp[u][1][j])) + bf16_value(dp[u][2][j]);
                        v += a2n[u][m][j] ? x : 0.f;
                    }
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
                if (g == 0) gb2[wave_id()][16 * m + i] += v;
            }
        }
        v8s d[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) d[c] = join(dp[0][c], dp[1][c]);
        const v8s dsel = (i & 3) == 0 ? d[0] : (i & 3) == 1 ? d[1] : d[2];
        const v8s none = {0, 0, 0, 0, 0, 0, 0, 0};
        const v8s d3 = i < 3 ? dsel : none, d2 = !far && i >= 4 && i < 7 ? dsel : none;
        v8s a1[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) a1[k] = join(a1n[0][k], a1n[1][k]);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const v8s a2 = join(a2n[0][m], a2n[1][m]);
            const v4i mask = nonzero(a2);
            const v8s unit = {kOne, kOne, kOne, kOne, kOne, kOne, kOne, kOne};
            gv[m] = mfma32(a2, d3, gv[m]);
            gv[m] = mfma32(masked(mask, unit), d2, gv[m]);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const v8s md = masked(mask, d[c]);
#pragma unroll
                for (int k = 0; k < 4; ++k) gw2[m][k] = mfma32(md, a1[k], gw2[m][k]);
            }
        }
    }
    // the workgroup's sums: its waves one after the other
#pragma unroll
    for (int o = 16; o < kWave; o <<= 1) {
        gb3 += __shfl_xor(gb3, o);
        loss += __shfl_xor(loss, o);
    }
    for (int w = 0; w < kBT / kWave; ++w) {
        if (wave_id() == w) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int h = 16 * m + 4 * g + j;
#pragma unroll
                    for (int k = 0; k < 4; ++k) sum[oW2 + h * kH + 16 * k + i] += gw2[m][k][j];
                    if (i < kFP) sum[oW1 + h * kFP + i] += gw1[m][j];
                    if (i == kFP) sum[oB1 + h] += gw1[m][j];
                    const float v = gv[m][j] + __shfl_down(gv[m][j], 1) + __shfl_down(gv[m][j], 2);
                    if (i == 0) sum[oW3 + h] += v;
                    if (i == 4) sum[oB2 + h] += v + gb2[w][h];
                }
            if (l == 0) {        // (every lane of a group holds the group's samples' values)
                sum[oB3] += gb3;
                lsum[w] = loss;
            }
        }
        __syncthreads();
    }
    float* pb = part + static_cast<int64_t>(blockIdx.x) * kNP;
    for (int e = t; e < kNP; e += kBT) {
        const int h = e >= oW2 && e < oB2 ? (e - oW2) / kH : e >= oB2 && e < oW3 ? e - oB2 : -1;
        pb[e] = h >= 0 ? sum[e] * bf16_round(P[oW3 + h]) : sum[e];
    }
    if (t == 0) loss_part[blockIdx.x] = ((lsum[0] + lsum[1]) + lsum[2]) + lsum[3];
}

// The gradient with float32 operands throughout (no rounding points), for
// checking it against a float64 reference: LDS tiles of 32 samples.
__global__ void __launch_bounds__(kBT) k_mlp_grad(const float* __restrict__ P, const float* __restrict__ feats,
                                                  const float* __restrict__ target, int64_t n, float inv_n,
                                                  float* __restrict__ part, double* __restrict__ loss_part) {
    __shared__ float W1q[kH * kFP], W2q[kH * kH], w3q[kH], b1[kH], b2[kH];
    __shared__ float X[kTS][kFP];
    __shared__ float Z1[kTS][kH], A1[kTS][kH], Z2[kTS][kH], D2[kTS][kH];
    __shared__ float dO[kTS];
    __shared__ double red[kBT / kWave];
    const int t = threadIdx.x;
    for (int e = t; e < kH * kFP; e += kBT) W1q[e] = P[oW1 + e];
    for (int e = t; e < kH * kH; e += kBT) W2q[e] = P[oW2 + e];
    if (t < kH) {
        w3q[t] = P[oW3 + t];
        b1[t] = P[oB1 + t];
        b2[t] = P[oB2 + t];
    }
    const float b3 = P[oB3];
    float gW2[16], gW1[2], gv = 0.f;     // gv: gb1 / gb2 / gw3 / gb3 entry of this thread
    for (int q = 0; q < 16; ++q) gW2[q] = 0.f;
    gW1[0] = gW1[1] = 0.f;
    double loss = 0;
    __syncthreads();
    const int64_t ntiles = (n + kTS - 1) / kTS;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += kGradGrid) {
        const int64_t s0 = tile * kTS;
        {
            int s = t / kFP, f = t % kFP;
            int64_t smp = s0 + s;
            X[s][f] = smp < n ? feats[smp * kFP + f] : 0.f;
        }
        __syncthreads();
        for (int q = 0; q < 8; ++q) {
            int e = t + kBT * q, s = e / kH, h = e % kH;
            float z = b1[h];
            for (int f = 0; f < kFP; ++f) z = __fmaf_rn(X[s][f], W1q[h * kFP + f], z);
            Z1[s][h] = z;
            A1[s][h] = (z > 0.f ? z : 0.f);
        }
        __syncthreads();
        for (int q = 0; q < 8; ++q) {
            int e = t + kBT * q, s = e / kH, h = e % kH;
            float z = b2[h];
            for (int k = 0; k < kH; ++k) z = __fmaf_rn(A1[s][k], W2q[h * kH + k], z);
            Z2[s][h] = z;
        }
        __syncthreads();
        if (t < kTS) {
            int64_t smp = s0 + t;
            float o = b3;
            for (int h = 0; h < kH; ++h) {
                float z = Z2[t][h];
                o = __fmaf_rn((z > 0.f ? z : 0.f), w3q[h], o);
            }
            if (smp < n) {
                float e = o - target[smp];
                loss += static_cast<double>(e) * e;
                dO[t] = 2.f * e * inv_n;
            } else {
                dO[t] = 0.f;
            }
        }
        __syncthreads();
        for (int q = 0; q < 8; ++q) {
            int e = t + kBT * q, s = e / kH, h = e % kH;
            D2[s][h] = Z2[s][h] > 0.f ? dO[s] * w3q[h] : 0.f;
        }
        __syncthreads();
        for (int q = 0; q < 16; ++q) {
            int e = t + kBT * q, h = e / kH, k = e % kH;
            float a = gW2[q];
            for (int s = 0; s < kTS; ++s) a = __fmaf_rn(D2[s][h], A1[s][k], a);
            gW2[q] = a;
        }
        if (t >= kH && t < 2 * kH) {
            for (int s = 0; s < kTS; ++s) gv += D2[s][t - kH];
        } else if (t >= 2 * kH && t < 3 * kH) {
            int h = t - 2 * kH;
            for (int s = 0; s < kTS; ++s) {
                float z = Z2[s][h];
                gv = __fmaf_rn(dO[s], (z > 0.f ? z : 0.f), gv);
            }
        } else if (t == 3 * kH) {
            for (int s = 0; s < kTS; ++s) gv += dO[s];
        }
        __syncthreads();
        // dz1 = (W2^T dz2) masked by z1 > 0, into Z2 (no longer needed)
        for (int q = 0; q < 8; ++q) {
            int e = t + kBT * q, s = e / kH, k = e % kH;
            float a = 0.f;
            for (int h = 0; h < kH; ++h) a = __fmaf_rn(D2[s][h], W2q[h * kH + k], a);
            Z2[s][k] = Z1[s][k] > 0.f ? a : 0.f;
        }
        __syncthreads();
        for (int q = 0; q < 2; ++q) {
            int e = t + kBT * q, h = e / kFP, f = e % kFP;
            float a = gW1[q];
            for (int s = 0; s < kTS; ++s) a = __fmaf_rn(Z2[s][h], X[s][f], a);
            gW1[q] = a;
        }
        if (t < kH)
            for (int s = 0; s < kTS; ++s) gv += Z2[s][t];
        __syncthreads();
    }
    float* pb = part + static_cast<int64_t>(blockIdx.x) * kNP;
    for (int q = 0; q < 16; ++q) pb[oW2 + t + kBT * q] = gW2[q];
    for (int q = 0; q < 2; ++q) pb[oW1 + t + kBT * q] = gW1[q];
    if (t < kH) pb[oB1 + t] = gv;
    else if (t < 2 * kH) pb[oB2 + t - kH] = gv;
    else if (t < 3 * kH) pb[oW3 + t - 2 * kH] = gv;
    else if (t == 3 * kH) pb[oB3] = gv;
    double ls = block_sum_f64<kBT>(loss, red);
    if (t == 0) loss_part[blockIdx.x] = ls;
}

// Sums the workgroups' partials in a fixed order: 16 interleaved slices of
// them per parameter, then the slices.  nb workgroups wrote partials.
constexpr int kFinalP = 64, kFinalS = 16;

__global__ void __launch_bounds__(kFinalP * kFinalS) k_mlp_grad_final(const float* __restrict__ part,
                                                                      const double* __restrict__ loss_part, int nb,
                                                                      double inv_n, float* __restrict__ grad,
                                                                      double* __restrict__ loss) {
    __shared__ float slice[kFinalS][kFinalP];
    const int p0 = blockIdx.x * kFinalP + threadIdx.x % kFinalP, p = p0 < kNP ? p0 : kNP - 1;
    const int q = threadIdx.x / kFinalP;
    float a = 0.f;
#pragma unroll 8
    for (int b = q; b < nb; b += kFinalS) a += part[static_cast<int64_t>(b) * kNP + p];
    slice[q][threadIdx.x % kFinalP] = a;
    __syncthreads();
    if (threadIdx.x < kFinalP && p0 < kNP) {
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < kFinalS; ++k) v += slice[k][threadIdx.x];
        grad[p0] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x / kWave == 1 && loss) {
        double s = 0;
        for (int b = lane_id(); b < nb; b += kWave) s += loss_part[b];
        s = wave_sum(s);
        if (lane_id() == 0) *loss = s * inv_n;
    }
}

__global__ void k_adam(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNP) return;
    float gp = g[p];
    float mp = b1 * m[p] + (1.f - b1) * gp;
    float vp = b2 * v[p] + (1.f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    P[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

template <int C>
void learned_c(Graph& g, const ahr_filter_spec& spec, const float* params, const float beta[4], const float* in,
               float* out, float* feats, float* hops, float* stats_out, hipStream_t s) {
    run_hops(g, spec, in, C, s);
    LearnArgs a;
    a.z0 = g.z0.p;
    a.z1 = g.zh[0].p;
    a.z2 = g.zh[1].p;
    a.z3 = g.zh[2].p;
    a.scale = g.scale.p;
    a.deg = g.deg.p;
    a.hsum = g.hsum.p;
    a.in = in;
    a.out = out;
    a.feats = feats;
    a.hops = hops;
    a.flags = g.nl.node_flags;
    a.perm = g.perm.p;
    a.params = params;
    for (int j = 0; j < 4; ++j) a.beta[j] = beta[j];
    a.n_inst = g.n_inst;
    a.write_out = out != nullptr;
    DevBuf<double> part;
    DevBuf<float> stats;
    DevBuf<float4> rowf;
    part.ensure(static_cast<size_t>(kStatGrid) * (3 * C + 1), s);
    stats.ensure(3 * C, s);
    rowf.ensure(static_cast<size_t>(g.n_inst) + 1, s);
    a.stats = stats.p;
    a.rowf = rowf.p;
    hipLaunchKernelGGL((k_colstat<C>), dim3(kStatGrid), dim3(kBT), 0, s, a, part.p);
    AHR_LAUNCHED("k_colstat");
    hipLaunchKernelGGL((k_colstat_final<C>), dim3(1), dim3(kBT), 0, s, a, part.p, stats.p);
    AHR_LAUNCHED("k_colstat_final");
    if (stats_out) AHR_HIP(hipMemcpyAsync(stats_out, stats.p, 3 * C * sizeof(float), hipMemcpyDeviceToDevice, s));
    {
        ProfScope ps(kStageMlp, s);
        // one resident set of workgroups, each wave walking its tiles with
        // the prefetch running: workgroups per CU at this kernel's occupancy
        // times the CUs
        const int64_t ntiles = (static_cast<int64_t>(g.n_inst) * C + 15) / 16;
        int dev = 0, cus = 0, per_cu = 0;
        AHR_HIP(hipGetDevice(&dev));
        AHR_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        AHR_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_learned<C>, kBT, 0));
        const int64_t resident = static_cast<int64_t>(cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
        const int64_t blocks = std::min<int64_t>((ntiles + 3) / 4, resident);
        hipLaunchKernelGGL((k_mlp_learned<C>), dim3(static_cast<unsigned>(blocks < 1 ? 1 : blocks)), dim3(kBT), 0, s,
                           a);
        AHR_LAUNCHED("k_mlp_learned");
    }
    if (feats) {
        const int64_t ns = static_cast<int64_t>(g.n_inst) * C;
        hipLaunchKernelGGL((k_feature_row<C>), dim3(grid_for(ns, kBT)), dim3(kBT), 0, s, a);
        AHR_LAUNCHED("k_feature_row");
    }
    part.release(s);
    stats.release(s);
    rowf.release(s);
}

}  // namespace

void run_learned(Graph& g, const ahr_filter_spec& spec, const float* params, const float beta[4], const float* in,
                 float* out, int32_t ncols, float* feats, float* hops, float* stats, hipStream_t s) {
    switch (ncols) {
        case 1: learned_c<1>(g, spec, params, beta, in, out, feats, hops, stats, s); break;
        case 2: learned_c<2>(g, spec, params, beta, in, out, feats, hops, stats, s); break;
        case 4: learned_c<4>(g, spec, params, beta, in, out, feats, hops, stats, s); break;
        case 8: learned_c<8>(g, spec, params, beta, in, out, feats, hops, stats, s); break;
        default: throw Error{AHR_EUNSUPPORTED, "ncols must be 1, 2, 4 or 8"};
    }
}

void mlp_forward(const float* params, const float* feats, int64_t n, float* o, hipStream_t s) {
    if (n <= 0) return;
    const int64_t ntiles = (n + 15) / 16;
    const int64_t blocks = std::min<int64_t>((ntiles + 3) / 4, 256 * 16);
    hipLaunchKernelGGL(k_mlp_forward, dim3(static_cast<unsigned>(blocks)), dim3(kBT), 0, s, params, feats, n, o);
    AHR_LAUNCHED("k_mlp_forward");
}

void mlp_loss_grad(const float* params, const float* feats, const float* target, int64_t n, float* grad,
                   double* loss, bool rounding, hipStream_t s) {
    DevBuf<float> part;
    DevBuf<double> lpart;
    // one wave per 32 samples until the grid is full
    const int64_t need = (n + 4 * kTS - 1) / (4 * kTS);
    const int nb = !rounding ? kGradGrid : static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(need, kGradMax)));
    part.ensure(static_cast<size_t>(nb) * kNP, s);
    lpart.ensure(nb, s);
    const float inv_n = n > 0 ? 1.f / static_cast<float>(n) : 0.f;
    hipLaunchKernelGGL((rounding ? k_mlp_grad_mfma : k_mlp_grad), dim3(nb), dim3(kBT), 0, s, params, feats, target, n,
                       inv_n, part.p, lpart.p);
    AHR_LAUNCHED("k_mlp_grad");
    hipLaunchKernelGGL(k_mlp_grad_final, dim3(grid_for(kNP, kFinalP)), dim3(kFinalP * kFinalS), 0, s, part.p, lpart.p,
                       nb, n > 0 ? 1.0 / static_cast<double>(n) : 0.0, grad, loss);
    AHR_LAUNCHED("k_mlp_grad_final");
    part.release(s);
    lpart.release(s);
}

void mlp_adam(float* params, float* m, float* v, const float* grad, int32_t step, float lr, float b1, float b2,
              float eps, hipStream_t s) {
    const float c1 = 1.f - powf(b1, static_cast<float>(step));
    const float c2 = 1.f - powf(b2, static_cast<float>(step));
    hipLaunchKernelGGL(k_adam, dim3(grid_for(kNP, kBT)), dim3(kBT), 0, s, params, m, v, grad, lr, b1, b2, eps, c1, c2);
    AHR_LAUNCHED("k_adam");
}

}  // namespace ahr
