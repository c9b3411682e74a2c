// bh_learned.hip -- data, labels and training kernels of the learned opening
// rule (not part of the paper; see bh_learned.hpp for the rule itself).
//
// Labels come from the method itself: for a candidate (group, node) pair the
// exact force of the node's particles on every particle of the group is
// summed directly in FP64 and compared with the node's monopole (the
// centre-of-mass approximation of Sec. 5.1); the label is the largest error
// over the group in units of G M / d^2, on the lg2p scale.
//
// Training is plain minibatch Adam on the mean squared error.  Gradients of
// a batch are summed per parameter over the batch in a fixed order, so a
// run is reproducible.
#include "bh_learned.hpp"

namespace {

constexpr int TPB = 256;

inline unsigned grid_for(size_t n, size_t cap = 8192) {
    size_t b = (n + TPB - 1) / TPB;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

__global__ void k_node_qn(DevState d) {
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nn; v += stride) {
        const uint32_t meta = d.nd_meta[v];
        const double S = (double)(1u << BH_MAXLEVEL) / d.box[meta_sys(meta)].w;   // root side, exact
        const double side = ldexp(S, -(int)meta_level(meta));
        d.nd_qn[v] = node_qn(d.nd_quad + (size_t)v * 6, d.nd_mom[v].w, side);
    }
}

// Self-gravity acceleration magnitude of each group (mean, or smallest, over
// its particles): the error budget scale of the learned rule.
__global__ void __launch_bounds__(TPB) k_group_amin(DevState d) {
    const uint32_t ng = d.cnt->n_groups;
    const uint32_t wpb = TPB / 64;
    for (uint32_t g = blockIdx.x * wpb + (threadIdx.x >> 6); g < ng; g += gridDim.x * wpb) {
        const double a = group_budget(d, d.grp[g]);
        if (__lane_id() == 0) d.g_amin[g] = a;
    }
}

// One workgroup per candidate pair: features and the exact label.
__global__ void __launch_bounds__(TPB) k_cand(DevState d, uint64_t n_cand, float4 *X, float *Y) {
    __shared__ double4 tile[TPB];
    __shared__ double red[TPB / 64];
    const uint32_t ng = d.cnt->n_groups, nn = d.cnt->lvl_off[BH_NLEVELS];
    for (uint64_t p = blockIdx.x; p < n_cand; p += gridDim.x) {
        const uint2 cv = d.cand[p];
        // every loop below is bounded by the pair's group size and node
        // count; a pair outside the tree or above the cap is not evaluated
        const bool bad = cv.x >= ng || cv.y >= nn || d.nd_count[cv.y] > d.count_cap ||
                         (uint64_t)d.grp[cv.x].begin + d.grp[cv.x].count > d.n ||
                         (uint64_t)d.nd_begin[cv.y] + d.nd_count[cv.y] > d.n;
        if (bad) {
            if (threadIdx.x == 0) {
                atomicOr(&d.cnt->flags[FLAG_CAND_BAD], 1u);
                X[p] = make_float4(0.f, 0.f, 0.f, 0.f);
                Y[p] = 0.f;
            }
            continue;
        }
        const GroupInfo gi = d.grp[cv.x];
        const uint32_t v = cv.y;
        const double4 mom = d.nd_mom[v];
        const int4 wr = d.nd_walk[v];
        const double r2 = box_ratio2(d.g_lo[cv.x], d.g_hi[cv.x], wr.x & 0xffffff, wr.y & 0xffffff, wr.z,
                                     (int)((uint32_t)wr.x >> 24));
        const double Msys = d.nd_mom[gi.sys].w;
        const PairGeom pg = pair_features(mom, r2, d.nd_qn[v], d.g_cen[cv.x], d.g_rad[cv.x], Msys);
        const uint32_t cb = d.nd_begin[v], cn = d.nd_count[v];
        double emax = 0.0;
        for (uint32_t i0 = 0; i0 < gi.count; i0 += TPB) {
            const uint32_t i = gi.begin + i0 + threadIdx.x;
            const bool on = i0 + threadIdx.x < gi.count;
            double xi = 0, yi = 0, zi = 0;
            if (on) {
                const double4 q = d.pos[i];
                xi = q.x;
                yi = q.y;
                zi = q.z;
            }
            double ex = 0, ey = 0, ez = 0;
            for (uint32_t j0 = 0; j0 < cn; j0 += TPB) {
                __syncthreads();
                if (j0 + threadIdx.x < cn) tile[threadIdx.x] = d.pos[cb + j0 + threadIdx.x];
                __syncthreads();
                const uint32_t m = min((uint32_t)TPB, cn - j0);
                for (uint32_t k = 0; k < m; ++k) {
                    const double4 s = tile[k];
                    const double dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
                    const double r2 = dx * dx + dy * dy + dz * dz + d.eps2;
                    const double f = s.w / (r2 * sqrt(r2));
                    ex += f * dx;
                    ey += f * dy;
                    ez += f * dz;
                }
            }
            if (on) {
                const double dx = mom.x - xi, dy = mom.y - yi, dz = mom.z - zi;
                const double r2 = dx * dx + dy * dy + dz * dz + d.eps2;
                const double f = mom.w / (r2 * sqrt(r2));
                const double ux = d.G * (f * dx - ex), uy = d.G * (f * dy - ey), uz = d.G * (f * dz - ez);
                emax = fmax(emax, sqrt(ux * ux + uy * uy + uz * uz));
            }
        }
        emax = wave_max(emax);
        __syncthreads();
        if (__lane_id() == 0) red[threadIdx.x >> 6] = emax;
        __syncthreads();
        if (threadIdx.x == 0) {
            double e = red[0];
            for (int k = 1; k < TPB / 64; ++k) e = fmax(e, red[k]);
            const double ratio = (e * pg.d2) / (d.G * mom.w);
            X[p] = make_float4(pg.f[0], pg.f[1], pg.f[2], pg.f[3]);
            Y[p] = (float)lg2p(ratio);
        }
    }
}

// ---------------------------------------------------------------- training
// Normalisation: mean and 1/std of each feature and of the label.  Sums in
// FP64 in a fixed order: STAT_BLOCKS blocks over the rows, then one block over
// their partial sums (one block alone took 543 us for 300,000 rows, a chain of
// 1,200 dependent loads per thread; in two launches 12 us).
constexpr int STAT_BLOCKS = 256;

__global__ void __launch_bounds__(TPB) k_stats_part(const float4 *X, const float *Y, uint64_t n, double *part) {
    __shared__ double red[TPB / 64][10];
    double s[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (uint64_t i = (uint64_t)blockIdx.x * TPB + threadIdx.x; i < n; i += (uint64_t)STAT_BLOCKS * TPB) {
        const float4 x = X[i];
        const double v[5] = {x.x, x.y, x.z, x.w, Y[i]};
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            s[k] += v[k];
            s[5 + k] += v[k] * v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const double t = wave_sum(s[k]);
        if (__lane_id() == 0) red[threadIdx.x >> 6][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < 10) {
        double t = 0;
        for (int w = 0; w < TPB / 64; ++w) t += red[w][threadIdx.x];
        part[blockIdx.x * 10 + threadIdx.x] = t;
    }
}

__global__ void __launch_bounds__(TPB) k_stats_final(const double *part, uint64_t n, float *w) {
    __shared__ double red[TPB / 64][10];
    static_assert(STAT_BLOCKS == TPB, "one partial per thread");
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const double t = wave_sum(part[threadIdx.x * 10 + k]);
        if (__lane_id() == 0) red[threadIdx.x >> 6][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        const int k = threadIdx.x;
        double S = 0, Q = 0;
        for (int v = 0; v < TPB / 64; ++v) {
            S += red[v][k];
            Q += red[v][5 + k];
        }
        const double mean = S / (double)n;
        double var = Q / (double)n - mean * mean;
        const double sd = var > 1e-24 ? sqrt(var) : 1.0;
        if (k < 4) {
            w[MLP_XMEAN + k] = (float)mean;
            w[MLP_XISTD + k] = (float)(1.0 / sd);
        } else {
            w[MLP_YMEAN] = (float)mean;
            w[MLP_YSTD] = (float)sd;
        }
    }
}

// Gradient of a batch.  A block takes 64 samples at a time through forward,
// backward and the sum over its samples without leaving the CU.  What bounds
// it is a chain of latencies: a batch of 4096 is 64 blocks, one per CU.  So
// everything that is a contraction runs on the matrix cores
// (v_mfma_f32_32x32x2_f32, 64 cycles for 2048 multiply-adds of one wave):
// waves 0 and 1 take 32 samples each, units by samples, through both layers
// forward and the second one backward, with the layouts of wave_net_forward;
// then they sum the 32 x 32 gradient of the second layer over their samples,
// while waves 2 and 3 take the other 225 sums, one or two per thread, from LDS
// (rows of 65 floats: lanes of one row and rows of one lane both fall in
// distinct banks).  At most GRAD_BLOCKS blocks, so that k_grad_final reads at
// most that many partial sums per parameter.  Forward and backward of a sample
// are chains of fmaf in ascending unit, as with one thread per sample.
// 4096 samples: one thread per parameter over the batch 969 + 30 us (sums,
// forward and backward); one lane per sample with scalar weight loads 12.6 us;
// now 10.8 us, some 8 of them launch, loads of rows and weights, and stores.
// 100 training steps of 4096 rows 101.3 -> 1.79 (lanes) -> 1.56 ms.
constexpr int GS = 64;              // samples per block and round
constexpr int GLD = GS + 1;         // LDS row of one unit over the samples
constexpr int GRAD_BLOCKS = 256;

__global__ void __launch_bounds__(TPB) k_grad_part(const float *w, const float4 *X, const float *Y,
                                                  const uint32_t *idx, uint32_t B, float *part, double *lossp) {
    __shared__ float xs[4][GLD], h1[MLP_NH][GLD], h2[MLP_NH][GLD], g1[MLP_NH][GLD], g2[MLP_NH][GLD], gos[GS];
    __shared__ float red[2][MLP_NH * MLP_NH];
    __shared__ double lred[2];
    __shared__ alignas(16) float s_net[WNET_LDS];
    const int t = threadIdx.x;
    const int lane = __lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool front = wv < 2;
    const int col = lane & 31, half = lane >> 5;
    const float *rest = s_net + WNET_REST;
    WaveNet net;
    float w2t[MLP_NH / 2];          // the second layer transposed, for the way back
    if (front) {
        net = wave_net_load(w);
#pragma unroll
        for (int s = 0; s < MLP_NH / 2; ++s) w2t[s] = w[MLP_W2 + (2 * s + half) * MLP_NH + col];
    }
    for (int k = t; k < WNET_LDS; k += TPB) s_net[k] = wave_net_lds_entry(w, k);
    // the sums outside W2: thread k of waves 2 and 3 has W1's entry k and one of the rest, operand rows a * b
    // (b null: a alone)
    const int k2 = t - 128;
    const float *ra = gos, *rb = nullptr;
    int dst = -1;
    if (k2 >= 0) {
        if (k2 < 32) {
            dst = MLP_B1 + k2;
            ra = g1[k2];
        } else if (k2 < 64) {
            dst = MLP_B2 + (k2 - 32);
            ra = g2[k2 - 32];
        } else if (k2 < 96) {
            dst = MLP_W3 + (k2 - 64);
            rb = h2[k2 - 64];
        } else if (k2 == 96) {
            dst = MLP_B3;
        }
    }
    float sum = 0.0f, sum1 = 0.0f;
    double loss = 0.0;
    mlp_f16 acc = {};
    const uint32_t rounds = (B + GS - 1) / GS;
    for (uint32_t c = blockIdx.x; c < rounds; c += gridDim.x) {
        const int n = 32 * wv + col;
        const uint32_t b = c * GS + n;
        const bool valid = front && b < B;
        const uint32_t i = valid ? (idx ? idx[b] : b) : 0u;
        const float4 xx = X[i];
        const float yy = Y[i];
        __syncthreads();                // s_net is there; the last round's sums are done
        if (front) {
            const float f[4] = {xx.x, xx.y, xx.z, xx.w};
            float x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float tt = f[k] - rest[1 + k];
                x[k] = valid ? tt * rest[1 + MLP_NIN + k] : 0.0f;   // columns past the batch add exact zeros
                if (half == 0) xs[k][n] = x[k];
            }
            mlp_f16 h, a;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int u = 8 * (r >> 2) + 4 * half + (r & 3);
                h[r] = s_net[u];
                a[r] = s_net[WNET_B2 + u];
            }
            h = __builtin_amdgcn_mfma_f32_32x32x2f32(net.w1[0], half ? x[1] : x[0], h, 0, 0, 0);
            h = __builtin_amdgcn_mfma_f32_32x32x2f32(net.w1[1], half ? x[3] : x[2], h, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                h[r] = h[r] > 0.0f ? h[r] : 0.0f;
                h1[8 * (r >> 2) + 4 * half + (r & 3)][n] = h[r];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4] = {h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]};
                a = wave_net_steps(net.w2 + 4 * q, v, a);
            }
            float out = rest[0];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float lo[4], hi[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int r = 4 * q + k;
                    a[r] = a[r] > 0.0f ? a[r] : 0.0f;
                    h2[8 * q + 4 * half + k][n] = a[r];
                    lo[k] = hi[k] = a[r];
                    swap_halves(lo[k], hi[k]);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) out = fmaf(s_net[WNET_W3 + 8 * q + k], lo[k], out);
#pragma unroll
                for (int k = 0; k < 4; ++k) out = fmaf(s_net[WNET_W3 + 8 * q + 4 + k], hi[k], out);
            }
            // loss on the normalised label: (out - (y - mean) / sd)^2, averaged over the batch
            const float yt = (yy - rest[1 + 2 * MLP_NIN]) / rest[2 + 2 * MLP_NIN];
            const float r = out - yt;
            const float go = valid ? 2.0f * r / (float)B : 0.0f;
            if (half == 0) {
                gos[n] = go;
                const float r2 = r * r;
                if (valid) loss += (double)r2;
            }
            mlp_f16 gk = {};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int u = 8 * q + 4 * half + k;
                    v[k] = a[4 * q + k] > 0.0f ? go * s_net[WNET_W3 + u] : 0.0f;
                    g2[u][n] = v[k];
                }
                gk = wave_net_steps(w2t + 4 * q, v, gk);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) g1[8 * (k >> 2) + 4 * half + (k & 3)][n] = h[k] > 0.0f ? gk[k] : 0.0f;
        }
        __syncthreads();
        if (front) {
            // W2: sum over this wave's 32 samples, two per instruction
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                const int sm = 32 * wv + 2 * st + half;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(g2[col][sm], h1[col][sm], acc, 0, 0, 0);
            }
        } else {
            const float *r1 = g1[k2 >> 2], *x1 = xs[k2 & 3];
#pragma unroll 8
            for (int sm = 0; sm < GS; ++sm) {
                sum1 = fmaf(r1[sm], x1[sm], sum1);
                sum = rb ? fmaf(ra[sm], rb[sm], sum) : sum + ra[sm];
            }
        }
    }
    if (front) {
        // matrix layout: element r of a lane is row 8 (r / 4) + r % 4 + 4 (lane / 32), column lane % 32
#pragma unroll
        for (int r = 0; r < 16; ++r) red[wv][(8 * (r >> 2) + (r & 3) + 4 * half) * MLP_NH + col] = acc[r];
        loss = wave_sum(loss);
        if (lane == 0) lred[wv] = loss;
    }
    __syncthreads();
    float *o = part + (size_t)blockIdx.x * MLP_NTRAIN;
    for (int e = t; e < MLP_NH * MLP_NH; e += TPB) o[MLP_W2 + e] = red[0][e] + red[1][e];
    if (!front) o[MLP_W1 + k2] = sum1;
    if (dst >= 0) o[dst] = sum;
    if (t == 0) lossp[blockIdx.x] = lred[0] + lred[1];
}

// Adam step of one parameter (Kingma & Ba 2015); c1, c2 = 1 - beta^t.
struct AdamArgs {
    float *w, *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_step(const AdamArgs &a, int p, float gp) {
    const float mp = a.b1 * a.m[p] + (1.0f - a.b1) * gp;
    const float vp = a.b2 * a.v[p] + (1.0f - a.b2) * gp * gp;
    a.m[p] = mp;
    a.v[p] = vp;
    a.w[p] -= a.lr * (mp / a.c1) / (sqrtf(vp / a.c2) + a.eps);
}

// The blocks' partial sums added in a fixed order, four threads per
// parameter; ADAM: the parameter's optimiser step in the same launch.
template <bool ADAM>
__global__ void __launch_bounds__(TPB) k_grad_final(const float *part, const double *lossp, int nb, uint32_t B,
                                                   float *grad, float *loss, AdamArgs ad) {
    __shared__ float red[4][64];
    const int q = threadIdx.x >> 6, lane = __lane_id();
    const int p = blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (p < MLP_NTRAIN) {
#pragma unroll 8
        for (int b = q; b < nb; b += 4) s += part[(size_t)b * MLP_NTRAIN + p];
    }
    red[q][lane] = s;
    __syncthreads();
    if (q == 0 && p < MLP_NTRAIN) {
        const float g = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
        if (ADAM) adam_step(ad, p, g);
        else grad[p] = g;
    }
    if (q == 1 && loss && blockIdx.x == 0) {
        double l = 0.0;
        for (int b = lane; b < nb; b += 64) l += lossp[b];
        l = wave_sum(l);
        if (lane == 0) *loss = (float)(l / B);
    }
}

__global__ void k_adam(AdamArgs ad, const float *g) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < MLP_NTRAIN) adam_step(ad, p, g[p]);
}

// Squared error of the network over a set, summed in FP64: per block, in a fixed order.
__global__ void __launch_bounds__(TPB) k_sq_error(const float *w, const float4 *X, const float *Y, uint64_t n,
                                                 double *part) {
    __shared__ double red[TPB / 64];
    __shared__ alignas(16) float s_net[WNET_LDS];
    const WaveNet net = wave_net_load(w);
    for (int k = threadIdx.x; k < WNET_LDS; k += TPB) s_net[k] = wave_net_lds_entry(w, k);
    __syncthreads();
    double s = 0.0;
    for (uint64_t b = (uint64_t)blockIdx.x * TPB; b < n; b += (uint64_t)gridDim.x * TPB) {
        const uint64_t i = b + threadIdx.x;
        const float4 x = i < n ? X[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float f[4] = {x.x, x.y, x.z, x.w};
        const float y = wave_net_forward(net, s_net, f);
        if (i < n) {
            const double e = (double)y - (double)Y[i];
            s += e * e;
        }
    }
    s = wave_sum(s);
    if (__lane_id() == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ void __launch_bounds__(TPB) k_eval(const float *w, const float4 *X, uint64_t n, float *out) {
    __shared__ alignas(16) float s_net[WNET_LDS];
    const WaveNet net = wave_net_load(w);
    for (int k = threadIdx.x; k < WNET_LDS; k += TPB) s_net[k] = wave_net_lds_entry(w, k);
    __syncthreads();
    for (uint64_t b = (uint64_t)blockIdx.x * TPB; b < n; b += (uint64_t)gridDim.x * TPB) {
        const uint64_t i = b + threadIdx.x;
        const float4 x = i < n ? X[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float f[4] = {x.x, x.y, x.z, x.w};
        const float y = wave_net_forward(net, s_net, f);
        if (i < n) out[i] = y;
    }
}

// splitmix64 of (seed, i): shuffle keys
__global__ void k_perm_keys(uint64_t *key, uint32_t *val, uint64_t n, uint64_t seed) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint64_t z = seed + 0x9e3779b97f4a7c15ull * (i + 1);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        key[i] = (z ^ (z >> 31)) >> 32;
        val[i] = (uint32_t)i;
    }
}

}  // namespace

namespace bhk {

void node_qn(const DevState &d, hipStream_t s) {
    k_node_qn<<<grid_for(d.node_cap, 4096), TPB, 0, s>>>(d);
}

void group_amin(const DevState &d, hipStream_t s) {
    k_group_amin<<<grid_for((size_t)d.n * 64 / 8, 8192), TPB, 0, s>>>(d);
}

void cand_features_labels(const DevState &d, uint64_t n_cand, float4 *X, float *Y, hipStream_t s) {
    if (n_cand == 0) return;
    unsigned blocks = (unsigned)(n_cand < 65536 ? n_cand : 65536);
    k_cand<<<blocks, TPB, 0, s>>>(d, n_cand, X, Y);
}

// Scratch of the training kernels: partial sums of the batch gradient and
// loss (GRAD_BLOCKS), of the normalisation and of the squared error.
size_t mlp_scratch_bytes() {
    return (size_t)GRAD_BLOCKS * (MLP_NTRAIN * sizeof(float) + sizeof(double)) +
           (size_t)STAT_BLOCKS * 10 * sizeof(double) + MSE_BLOCKS * sizeof(double);
}

namespace {
struct Scratch {
    double *loss, *stat, *mse;
    float *part;
    explicit Scratch(void *p)
        : loss((double *)p), stat(loss + GRAD_BLOCKS), mse(stat + STAT_BLOCKS * 10), part((float *)(mse + MSE_BLOCKS)) {}
};
AdamArgs adam_args(const Adam &a) {
    return AdamArgs{a.w, a.m, a.v, a.lr, a.b1, a.b2, a.eps, 1.0f - powf(a.b1, (float)a.step),
                    1.0f - powf(a.b2, (float)a.step)};
}
}  // namespace

void mlp_stats(const float4 *X, const float *Y, uint64_t n, float *w, void *scratch, hipStream_t s) {
    const Scratch sc(scratch);
    k_stats_part<<<STAT_BLOCKS, TPB, 0, s>>>(X, Y, n, sc.stat);
    k_stats_final<<<1, TPB, 0, s>>>(sc.stat, n, w);
}

void mlp_batch_grad(const float *w, const float4 *X, const float *Y, const uint32_t *idx, uint32_t B, void *scratch,
                    float *grad, float *loss, const Adam *adam, hipStream_t s) {
    const Scratch sc(scratch);
    const uint32_t rounds = (B + GS - 1) / GS;
    const int nb = (int)(rounds < (uint32_t)GRAD_BLOCKS ? rounds : (uint32_t)GRAD_BLOCKS);
    k_grad_part<<<nb, TPB, 0, s>>>(w, X, Y, idx, B, sc.part, sc.loss);
    const unsigned blocks = (MLP_NTRAIN + 63) / 64;
    if (adam)
        k_grad_final<true><<<blocks, TPB, 0, s>>>(sc.part, sc.loss, nb, B, nullptr, nullptr, adam_args(*adam));
    else
        k_grad_final<false><<<blocks, TPB, 0, s>>>(sc.part, sc.loss, nb, B, grad, loss, AdamArgs{});
}

void mlp_adam(const Adam &a, const float *grad, hipStream_t s) {
    k_adam<<<(MLP_NTRAIN + 255) / 256, 256, 0, s>>>(adam_args(a), grad);
}

const double *mlp_sq_error(const float *w, const float4 *X, const float *Y, uint64_t n, void *scratch, hipStream_t s) {
    const Scratch sc(scratch);
    k_sq_error<<<MSE_BLOCKS, TPB, 0, s>>>(w, X, Y, n, sc.mse);
    return sc.mse;
}

void mlp_eval(const float *w, const float4 *X, uint64_t n, float *out, hipStream_t s) {
    if (n == 0) return;
    k_eval<<<grid_for(n), TPB, 0, s>>>(w, X, n, out);
}

void perm_keys(uint64_t *key, uint32_t *val, uint64_t n, uint64_t seed, hipStream_t s) {
    k_perm_keys<<<grid_for(n), TPB, 0, s>>>(key, val, n, seed);
}

}  // namespace bhk
