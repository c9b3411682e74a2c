// bh_direct.hip -- FP64 direct summation over all particles for a set of
// target particles: the exact sum that the tree method approximates
// (Sec. 4.2 (3d) applied with every node opened), used to judge the error
// of the Barnes-Hut forces.  With a collision radius every pair follows
// Eq. (2) with both branches (all sources are particles here).
//
// Grid: (target blocks of 64, source chunks).  Each workgroup stages 256
// sources at a time in LDS; its four waves take a quarter each against the
// same 64 targets; wave partials are added in a fixed order and written per
// source chunk, and a second kernel adds the chunks in order.  Gravity
// (scaled by G at the end) and contact terms are summed separately.
//
// What bounds it is FP64 issue, and through it the card's power: the clock is
// at 2.03 of 2.4 GHz.  A pair is 16 instructions of four cycles each and
// v_rsq_f64 (sixteen); a correctly rounded square root and division were 15
// more.  cube_inverse() below has none of their range handling, so every tile
// is checked while it is staged, and one that could leave its range (a
// coordinate or mass of 2^339 or more, infinite or NaN), or a softening length
// of 2^340 or more, takes them as before.
// 4096 targets against 2^20 sources: 7.45 -> 2.95 ms; loops unrolled 1 to 8
// times at 5 to 8 waves per SIMD are within 1%.  1000 targets of 60000: 2.70
// -> 0.073 ms, by the smaller chunks (chosen in launch()).  Each tile's 64
// pairs of a wave are summed apart before they join the lane's sum, which
// takes the rounding of long sums down: error against exact sums 2.4e-15 ->
// 5.8e-16 (relative 2-norm) at 2^20 sources.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "bh_internal.hpp"

namespace {

constexpr int DT = 256;
constexpr int DCHUNKS = 64;
constexpr int NC = 6;   // per (chunk, target) at most: gravity x, y, z, contact x, y, z

// Partial sums of the allocation-free direct sum (bh_direct_sum_static):
// room for DIRECT_STATIC_MAX_TARGETS targets at the largest chunk count,
// 12 MiB, one copy on every GPU the library runs on, held until the process
// ends.  Host code never passes this name to a kernel: it is a host-side
// stand-in; the device address comes from hipGetSymbolAddress, per device.
constexpr int64_t DIRECT_STATIC_MAX_TARGETS = 4096;
static __device__ __align__(256) double scratch[(size_t)DCHUNKS * DIRECT_STATIC_MAX_TARGETS * NC];

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
double *scratch_dev[MAX_DEVICES] = {};

// coordinates and masses from WIDE on, and any eps^2 from WIDE_EPS2 on, take the exact pair: below them
// r^2 < 2^682 and the exact pair's r^3 is finite, so that both pairs give a term or none alike
constexpr double WIDE = 0x1p339, WIDE_EPS2 = 0x1p680;
constexpr double TIGHT = 0x1p-300;       // and so do squared distances below

// m x^(-3/2) for TIGHT <= x < 2^682: the hardware estimate y of x^(-1/2) (relative
// error below 2^-24) and e = 1 - x y^2 give it as m y^3 (1 + 3/2 e + 15/8 e^2 + ...),
// the next term below 2^-67.  A rounding d of y^2 enters y^3 as d and the
// correction as -3/2 d: four roundings, one of them halved, against the three
// of a square root, a product and a division.
// (c15, c1875 are 3/2 and 15/8 in registers: literals are moved there for each pair.)
__device__ __forceinline__ double cube_inverse(double m, double x, double c15, double c1875) {
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double e = fma(-x, y2, 1.0);
    const double f = (m * y) * y2;
    return fma(f, e * fma(c1875, e, c15), f);
}

// SOFT: eps2 >= TIGHT, so that no pair is closer
template <bool COLL, bool SOFT>
__global__ void __launch_bounds__(DT) k_direct_part(const double *x, const double *y, const double *z,
                                                   const double *m, int64_t n, const int64_t *targets,
                                                   int64_t nt, double eps2, bhk::Contact ct, double *part,
                                                   int chunks) {
    __shared__ double4 tile[DT];
    __shared__ double red[NC][4][64];
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    const bool ton = t < nt;
    int64_t i = 0;
    double xi = 0, yi = 0, zi = 0;
    bool bad = false;             // a target index outside [0, n): NaN result, nothing read out of range
    if (ton) {
        i = targets[t];
        bad = i < 0 || i >= n;
        if (bad) i = 0;
        xi = x[i];
        yi = y[i];
        zi = z[i];
    }
    const double rc2 = ct.rc * ct.rc;
    const double rce2 = rc2 + eps2;
    const double rce = sqrt(rce2);
    const int64_t per = (n + chunks - 1) / chunks;
    const int64_t j0 = (int64_t)blockIdx.y * per, j1 = (j0 + per < n) ? j0 + per : n;
    double c15 = 1.5, c1875 = 1.875;
    asm volatile("" : "+v"(c15), "+s"(c1875));
    const bool far_i = !(fabs(xi) < WIDE && fabs(yi) < WIDE && fabs(zi) < WIDE);
    double ax = 0, ay = 0, az = 0, cx = 0, cy = 0, cz = 0;
    for (int64_t b = j0; b < j1; b += DT) {
        const int64_t j = b + threadIdx.x;
        bool wide = !(eps2 < WIDE_EPS2);
        if (j < j1) {
            const double4 s = make_double4(x[j], y[j], z[j], m[j]);
            tile[threadIdx.x] = s;
            wide = wide || !(fabs(s.x) < WIDE && fabs(s.y) < WIDE && fabs(s.z) < WIDE && fabs(s.w) < WIDE);
        }
        // a far target decides for its own lane: the others' bits do not depend on it
        const bool exact = __syncthreads_or(wide) || far_i;
        const int cnt = (int)((j1 - b < DT) ? j1 - b : DT);
        const int q0 = cnt * w / 4, q1 = cnt * (w + 1) / 4;
        double tx = 0, ty = 0, tz = 0;
        auto pair = [&](int k, auto in_range) {
            const double4 s = tile[k];
            const double dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
            const double d2 = dx * dx + dy * dy + dz * dz;
            if (COLL && d2 <= rc2) {
                if (d2 == 0.0 || !ton) return;
                // contact: gravity frozen on the contact sphere, spring and dashpot
                const double f = s.w / (rce2 * rce);
                tx += f * dx;
                ty += f * dy;
                tz += f * dz;
                const int64_t jj = b + k;
                const double dvx = ct.vx[jj] - ct.vx[i], dvy = ct.vy[jj] - ct.vy[i], dvz = ct.vz[jj] - ct.vz[i];
                const double r = sqrt(d2);
                const double rv = dx * dvx + dy * dvy + dz * dvz;
                const double fc = s.w / (m[i] + s.w) * (ct.kappa * (r - ct.rc) / r + ct.eta * rv / d2);
                cx += fc * dx;
                cy += fc * dy;
                cz += fc * dz;
                return;
            }
            const double r2 = COLL ? d2 + eps2 : fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
            double f;
            if (in_range && (SOFT || r2 >= TIGHT)) {
                f = cube_inverse(s.w, r2, c15, c1875);
            } else {
                if (r2 == 0.0) return;
                f = s.w / (r2 * sqrt(r2));
            }
            tx += f * dx;
            ty += f * dy;
            tz += f * dz;
        };
        if (exact) {
            for (int k = q0; k < q1; ++k) pair(k, std::false_type{});
        } else {
#pragma unroll 4
            for (int k = q0; k < q1; ++k) pair(k, std::true_type{});
        }
        ax += tx;
        ay += ty;
        az += tz;
        __syncthreads();
    }
    red[0][w][lane] = ax;
    red[1][w][lane] = ay;
    red[2][w][lane] = az;
    red[3][w][lane] = cx;
    red[4][w][lane] = cy;
    red[5][w][lane] = cz;
    __syncthreads();
    if (w == 0 && ton) {
        constexpr int C = COLL ? NC : 3;
        double *o = part + (size_t)blockIdx.y * C * nt + t;
        for (int a = 0; a < C; ++a)
            o[a * nt] = bad ? NAN : ((red[a][0][lane] + red[a][1][lane]) + red[a][2][lane]) + red[a][3][lane];
    }
}

template <bool COLL>
__global__ void k_direct_sum(const double *part, int64_t nt, int chunks, double G, double *ax, double *ay,
                             double *az) {
    constexpr int C = COLL ? NC : 3;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    double s[NC] = {0, 0, 0, 0, 0, 0};
#pragma unroll 8
    for (int c = 0; c < chunks; ++c)
        for (int a = 0; a < C; ++a) s[a] += part[((size_t)c * C + a) * nt + t];
    ax[t] = G * s[0] + s[3];
    ay[t] = G * s[1] + s[4];
    az[t] = G * s[2] + s[5];
}

template <bool COLL>
void launch(const double *x, const double *y, const double *z, const double *m, int64_t n, const int64_t *targets,
            int64_t nt, double eps2, double G, const bhk::Contact &ct, double *ax, double *ay, double *az,
            double *part, hipStream_t s) {
    // chunks of at least 1024 sources (four tiles), so that few targets or few
    // sources still make many workgroups; a rule of n alone: a target's sum
    // does not depend on the others asked for with it
    const int chunks = (int)std::min<int64_t>(DCHUNKS, std::max<int64_t>(1, (n + 1023) / 1024));
    const dim3 grid((unsigned)((nt + 63) / 64), (unsigned)chunks);
    if (eps2 >= TIGHT)
        k_direct_part<COLL, true><<<grid, DT, 0, s>>>(x, y, z, m, n, targets, nt, eps2, ct, part, chunks);
    else
        k_direct_part<COLL, false><<<grid, DT, 0, s>>>(x, y, z, m, n, targets, nt, eps2, ct, part, chunks);
    k_direct_sum<COLL><<<(unsigned)((nt + 63) / 64), 64, 0, s>>>(part, nt, chunks, G, ax, ay, az);
}

}  // namespace

namespace bhk {

int64_t direct_static_max_targets() { return DIRECT_STATIC_MAX_TARGETS; }

hipError_t direct_static_init(int device) {
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_dev[device]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;      // the device must be current
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_dev[device] = static_cast<double *>(p);
    return hipSuccess;
}

double *direct_static_scratch(int device) {
    if (device < 0 || device >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mu);
    return scratch_dev[device];
}

size_t direct_scratch_bytes(int64_t n_targets) {
    return (size_t)DCHUNKS * (size_t)n_targets * NC * sizeof(double);
}

void direct_sum(const double *x, const double *y, const double *z, const double *m, int64_t n,
                const int64_t *targets, int64_t nt, double eps2, double G, const Contact *contact, double *ax,
                double *ay, double *az, double *scratch, hipStream_t s) {
    if (contact)
        launch<true>(x, y, z, m, n, targets, nt, eps2, G, *contact, ax, ay, az, scratch, s);
    else
        launch<false>(x, y, z, m, n, targets, nt, eps2, G, Contact{0, 0, 0, nullptr, nullptr, nullptr}, ax, ay, az,
                      scratch, s);
}

}  // namespace bhk
