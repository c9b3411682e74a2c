// bh_learned.hpp -- device functions of the learned opening rule (not part of
// the paper; the paper's walk uses a fixed geometric rule).  Shared by the
// walk (inference), the feature kernel and the training kernels so that the
// three compute identical values.
//
// Rule: for a (group, node) pair with theta_min <= side/distance < theta_max
// (the geometric test of the walk at two angles), a 4-32-32-1 ReLU network
// predicts y = lg(monopole error of the node over the group /
// (G M / d^2)); the node is accepted when y < lg(tau * A_g * d^2 / (G M)),
// i.e. when the predicted error is below tau times the mean self-gravity
// acceleration A_g of the group's particles (from the last evaluation).  A single-particle node is exact and always
// accepted; nodes above the count cap fall back to the geometric theta.
//
// Every quantity that decides an acceptance is computed with correctly
// rounded operations in a fixed order (FP64 features, FP32 network with
// explicit fmaf, comparisons in FP64), so the decision is reproducible
// bit for bit by any implementation that follows the same order.
#pragma once
#include "bh_internal.hpp"

#define MLP_NIN 4
#define MLP_NH 32
#define MLP_W1 0                                   // [32][4]
#define MLP_B1 (MLP_W1 + MLP_NH * MLP_NIN)          // 128
#define MLP_W2 (MLP_B1 + MLP_NH)                    // 160, [32][32]
#define MLP_B2 (MLP_W2 + MLP_NH * MLP_NH)           // 1184
#define MLP_W3 (MLP_B2 + MLP_NH)                    // 1216
#define MLP_B3 (MLP_W3 + MLP_NH)                    // 1248
#define MLP_NTRAIN (MLP_B3 + 1)                     // 1249 trained parameters
#define MLP_XMEAN MLP_NTRAIN                        // 1249..1252
#define MLP_XISTD (MLP_XMEAN + MLP_NIN)             // 1253..1256
#define MLP_YMEAN (MLP_XISTD + MLP_NIN)             // 1257
#define MLP_YSTD (MLP_YMEAN + 1)                    // 1258
#define MLP_NPARAM (MLP_YSTD + 1)                   // 1259

// Piecewise-linear base-2 logarithm: x = m 2^e with m in [0.5, 1) gives
// e - 1 + (2m - 1); exact at powers of two, monotone, continuous, computed
// with one rounding.  0 maps to -1100, +inf to +1100.
__host__ __device__ __forceinline__ double lg2p(double x) {
    if (!(x > 0.0)) return -1100.0;
    if (x > 1.7976931348623157e308) return 1100.0;
    int e = 0;
    double m = frexp(x, &e);
    return (double)e + ((2.0 * m) - 2.0);
}

// Second-moment feature of a node: |Q|_F / (M s^2), Q the second moment
// about the centre of mass (xx, xy, xz, yy, yz, zz).
__device__ __forceinline__ float node_qn(const double *Q, double M, double s) {
    double qq = Q[0] * Q[0] + Q[3] * Q[3] + Q[5] * Q[5] + 2.0 * (Q[1] * Q[1]) + 2.0 * (Q[2] * Q[2]) +
                2.0 * (Q[4] * Q[4]);
    return (float)(sqrt(qq) / (M * (s * s)));
}

struct PairGeom {
    double d2;        // |com - group centre|^2
    float f[MLP_NIN];
};

// (side / distance from the node's centre to the group box)^2 in doubled
// integer grid units: the quantity the geometric opening test compares with
// theta^2.  The node must lie outside the box (distance > 0).
__device__ __forceinline__ double box_ratio2(int4 glo, int4 ghi, int Lx, int Ly, int Lz, int level) {
    const int64_t s = (int64_t)1 << (BH_MAXLEVEL - level);
    const int64_t L[3] = {Lx, Ly, Lz};
    const int64_t gl[3] = {glo.x, glo.y, glo.z}, gh[3] = {ghi.x, ghi.y, ghi.z};
    int64_t d2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t C = 2 * L[a] + s;
        int64_t da = 0;
        da = (2 * gl[a] - C > da) ? 2 * gl[a] - C : da;
        da = (C - 2 * gh[a] > da) ? C - 2 * gh[a] : da;
        d2 += da * da;
    }
    return (double)((2 * s) * (2 * s)) / (double)d2;
}

// Features of node (com, M, qn, box ratio r2 = box_ratio2) for a group
// (centre, half-diagonal rg) of a system of total mass Msys, all on the lg2p
// scale: the leading monopole error on the group's nearest particle relative
// to G M / d^2 behaves like qn r2 (d/d_box)^2, which is close to linear in
// these coordinates.
__device__ __forceinline__ PairGeom pair_features(double4 com, double r2, float qn, double4 gc, double rg,
                                                  double Msys) {
    PairGeom p;
    const double dx = com.x - gc.x, dy = com.y - gc.y, dz = com.z - gc.z;
    p.d2 = dx * dx + dy * dy + dz * dz;
    const double d = sqrt(p.d2);
    p.f[0] = (float)lg2p(r2);
    p.f[1] = (float)lg2p(rg / d);
    p.f[2] = (float)lg2p(com.w / Msys);
    p.f[3] = (float)lg2p((double)qn);
    return p;
}

// The value that the network's output is compared with, for a node in the band:
// accepted when the output is below it.
__device__ __forceinline__ double accept_below(const PairGeom &p, double M, double A_g, double tau, double G) {
    return lg2p(((tau * A_g) * p.d2) / (G * M));
}

// Network output in label units (lg of the relative monopole error) for 64
// inputs at once, one per lane of a full wave, on the matrix cores.  Each sum
// is a chain of fmaf in ascending input from its bias:
// v_mfma_f32_32x32x2_f32 adds its two products to the accumulator as two fused
// multiply-adds in ascending k (checked bit for bit against fmaf, subnormals
// included), so the output has the bits of that chain.  Layer weights sit in
// registers, loaded once per wave (lane l holds row l % 32 and column
// 2 s + l / 32 of step s); a D tile has its unit 8 q + 4 (l / 32) + i in
// register 4 q + i, and v_permlane32_swap of registers with neighbouring units
// gives the next layer's B operands, units in order.  One lane per input with
// the weights from memory was bound by them: some 340 loads per 64 nodes of a walk,
// 72% of the waves' time spent waiting.  Walk of 2^19 particles: 1581 -> 455
// us in 1914 groups; whole steps 33.6 -> 13.4 ms with groups of up to 64, 47.7
// -> 25.6 ms at 2^21 particles.
struct WaveNet {
    float w1[2], w2[MLP_NH / 2];
};

typedef float mlp_f16 __attribute__((ext_vector_type(16)));

// The weights outside the matrix operands, as the walk's blocks keep them in
// LDS: b1, b2, w3 (32 each), then b3, mean and 1/std of the inputs, of the label.
#define WNET_B2 MLP_NH
#define WNET_W3 (2 * MLP_NH)
#define WNET_REST (3 * MLP_NH)
#define WNET_LDS (WNET_REST + 1 + 2 * MLP_NIN + 2)

__device__ __forceinline__ float wave_net_lds_entry(const float *w, int k) {
    return k < WNET_B2     ? w[MLP_B1 + k]
           : k < WNET_W3   ? w[MLP_B2 + (k - WNET_B2)]
           : k < WNET_REST ? w[MLP_W3 + (k - WNET_W3)]
                           : w[MLP_B3 + (k - WNET_REST)];
}

__device__ __forceinline__ WaveNet wave_net_load(const float *w) {
    const int row = __lane_id() & 31, half = __lane_id() >> 5;
    WaveNet n;
#pragma unroll
    for (int s = 0; s < 2; ++s) n.w1[s] = w[MLP_W1 + row * MLP_NIN + 2 * s + half];
#pragma unroll
    for (int s = 0; s < MLP_NH / 2; ++s) n.w2[s] = w[MLP_W2 + row * MLP_NH + 2 * s + half];
    return n;
}

// a's upper 32 lanes against b's lower 32: (a.lo, b.lo) and (a.hi, b.hi)
__device__ __forceinline__ void swap_halves(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// Eight units of a D tile (registers 4 q .. 4 q + 3 of every lane) times their four steps of a layer.
__device__ __forceinline__ mlp_f16 wave_net_steps(const float *w, float v[4], mlp_f16 a) {
    swap_halves(v[0], v[1]);
    swap_halves(v[2], v[3]);
    a = __builtin_amdgcn_mfma_f32_32x32x2f32(w[0], v[0], a, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_32x32x2f32(w[1], v[2], a, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_32x32x2f32(w[2], v[1], a, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x2f32(w[3], v[3], a, 0, 0, 0);
}

// All 64 lanes call it together (an unused lane may hold any input).  c: the block's LDS copy (WNET_LDS floats, 16-byte aligned).
__device__ __forceinline__ float wave_net_forward(const WaveNet &n, const float *c, const float f[MLP_NIN]) {
    const int half4 = 4 * (__lane_id() >> 5);
    const float *rest = c + WNET_REST;
    float x[MLP_NIN];
#pragma unroll
    for (int k = 0; k < MLP_NIN; ++k) {
        const float t = f[k] - rest[1 + k];
        x[k] = t * rest[1 + MLP_NIN + k];
    }
    // B operands: x[0], x[2] those of lanes 0..31 (tile 0), x[1], x[3] those of lanes 32..63 (tile 1)
    swap_halves(x[0], x[1]);
    swap_halves(x[2], x[3]);
    mlp_f16 h[2], a[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) h[0][r] = h[1][r] = c[8 * (r >> 2) + half4 + (r & 3)];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[0][r] = a[1][r] = c[WNET_B2 + 8 * (r >> 2) + half4 + (r & 3)];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        h[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(n.w1[0], x[t], h[t], 0, 0, 0);
        h[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(n.w1[1], x[2 + t], h[t], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = h[t][4 * q + i] > 0.0f ? h[t][4 * q + i] : 0.0f;
            a[t] = wave_net_steps(n.w2 + 4 * q, v, a[t]);
        }
    }
    // a lane's own node: its units 8 q + i and 8 q + 4 + i
    float out = rest[0];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[i] = a[0][4 * q + i];
            hi[i] = a[1][4 * q + i];
            swap_halves(lo[i], hi[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) out = fmaf(c[WNET_W3 + 8 * q + i], lo[i] > 0.0f ? lo[i] : 0.0f, out);
#pragma unroll
        for (int i = 0; i < 4; ++i) out = fmaf(c[WNET_W3 + 8 * q + 4 + i], hi[i] > 0.0f ? hi[i] : 0.0f, out);
    }
    return fmaf(out, rest[1 + 2 * MLP_NIN + 1], rest[1 + 2 * MLP_NIN]);
}
