// bh_force.hip -- the interaction double loop of Iwasawa et al. (2019)
// Sec. 4.2 step (3d): for every group, every particle of the group against
// every entry of the group's lists.  The pair term is the gravity branch of
// Eq. (2) with Plummer softening,
//     a_i += G m_j (x_j - x_i) / (|x_j - x_i|^2 + eps^2)^(3/2),
// nodes acting as point masses at their centre of mass (Sec. 5.1).
//
// Precision (Sec. 4.7, shifted origin): in the FP32 variant the positions
// of the group's particles and of every source are taken relative to the
// group centre in FP64 and only then rounded to FP32; the pair terms and
// their sums are FP32, the result is scaled by G and written in FP64.  The
// FP64 variant is the same loop in double precision.  In FP32, a system
// whose particles all have one mass m0 (the paper's ring particles) enters
// the particle-pair loop with unit masses and its node masses in units of
// m0, the sums being scaled by G m0 at the end: one multiply fewer per pair.
//
// Sources are staged 512 at a time (the FP32 gravity-only kernels also come
// with tiles of 256, a choice of the autotuner) in LDS as group-relative
// float4 (x, y, z, m); particle-list leaves are read 256 at a time, a prefix sum over their
// sizes places their particles in the tiles, and the FP32 gravity-only
// kernels list the chunk's particle ids in LDS once so that staging a source
// is one LDS read (a chunk of more than 2048 particles, possible only with
// big level-21 leaves, searches the leaf offsets instead).  Inside a leapfrog
// step these kernels also apply the closing half kick to each particle.
//
// Scheduling (Sec. 4.6): a persistent grid takes groups, 256 particles at a
// time, from an atomic queue in order of decreasing interaction count, so the longest lists start
// first and the tail is made of short ones.  All four waves of a workgroup
// share one LDS tile of sources (the paper's cores sharing a cache on one
// list).  The waves take 64-particle chunks of the group, the waves left
// over splitting the source range.  A partial chunk -- a small group, or the
// last chunk of a larger one -- keeps most of its lanes busy.  In FP64 the
// wave takes as many sub-slices of the source range as the chunk's particles
// fit into it, up to 8.  In FP32 at most 8, 16 or
// 25..32 particles spread the wave over 8, 4 or 2 sub-slices of the source
// range; 17..24, 33..40 and 49..56 particles (3, 5, 7 slices of 8) run in
// eighths mode and 41..48 in tail mode, where the lanes without particles
// take the last parts of the range for the particles' slices in turn (the
// tile is padded with massless sources so that every part has one length).
// Partial sums are added in a fixed order, so results do not depend on
// timing.
//
// Collision branch of Eq. (2) (particle sources only, when rc > 0): inside
// the pair loop the squared distance is clamped from below at rc^2 + eps^2,
// which is exactly the branch's gravity part (continuous at rc, so the FP32
// clamp needs no exact decision), and each lane keeps the smallest squared
// distance it met.  A wave in which some lane came within a bound that the
// FP32 rounding of the relative coordinates cannot cross runs a second pass
// over the same tile, for the candidates only: the contact decision
// dx*dx + dy*dy + dz*dz <= rc^2 and the spring and dashpot terms are taken
// in FP64 from the absolute positions and velocities, and summed in FP64
// apart from the gravity sums.  Particle tiles thus run the 13-instruction
// body plus a max and a min; node tiles run the plain loop.  These kernels
// use the sub-slices only (no tail or eighths mode, no id list, no
// fused kick: their LDS and registers are at the six-workgroup limit, and the
// dashpot reads other particles' velocities).
#include <algorithm>

#include "bh_internal.hpp"

namespace {

constexpr int FT = 256;      // threads per workgroup (4 waves)
static_assert(FT == ITEM_PARTICLES, "a workgroup takes an item's particles at once");
constexpr int TJ_MAX = 512;  // sources per LDS tile at most (two per thread); 256 is the other tile
constexpr int LC = FT;       // particle-list leaves per chunk (one per thread)
constexpr int PIDX = 2048;   // particle ids of a leaf chunk listed in LDS (FP32 gravity-only kernels)

template <typename R> struct V4;
template <> struct V4<float> { using T = float4; };
template <> struct V4<double> { using T = double4; };

template <typename R>
__device__ __forceinline__ typename V4<R>::T mk4(R a, R b, R c, R e);
template <>
__device__ __forceinline__ float4 mk4<float>(float a, float b, float c, float e) { return make_float4(a, b, c, e); }
template <>
__device__ __forceinline__ double4 mk4<double>(double a, double b, double c, double e) {
    return make_double4(a, b, c, e);
}

template <typename R>
__device__ __forceinline__ R rsqrt_r(R x);
template <>
__device__ __forceinline__ float rsqrt_r<float>(float x) { return __builtin_amdgcn_rsqf(x); }
// FP64: the hardware estimate (relative error below 2^-24 on gfx950, measured
// over 1e-20..1e20) refined by one Newton step for y = x^(-1/2),
// y <- y + (y/2)(1 - x y^2), which squares the error (below 5e-15 measured):
// far inside the FP64 bar, at a fraction of a division and a square root.
template <>
__device__ __forceinline__ double rsqrt_r<double>(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

template <typename R>
__device__ __forceinline__ R fma_r(R a, R b, R c);
template <>
__device__ __forceinline__ float fma_r<float>(float a, float b, float c) { return fmaf(a, b, c); }
template <>
__device__ __forceinline__ double fma_r<double>(double a, double b, double c) { return fma(a, b, c); }

// The FP32 gravity pair loop over 4 n4 sources from LDS address `addr` (per
// lane), in the order and with the roundings of the C++ loops below.
//
// What bounds it is instruction issue (measured on gfx950, wave64, 24 waves per
// CU; cycles per instruction and SIMD at 2.4 GHz):
//   - A VALU instruction on VGPRs issues in 2.3 to 2.5 cycles, but registers
//     lie in two banks, even and odd: instructions that keep reading one bank
//     (fma x, x, y with both even) take 3.6 to 4.2.  An SGPR operand always
//     costs 4.2 to 4.4.  v_rsq_f32 takes 8.2 and overlaps nothing.
//   - In the compiler's loop four of eight sources wait for their LDS read in
//     full, and a loop that starts away from a 64-byte line loses up to 10%.
// So the loop is aligned, names its registers (the map is the best of 1500
// tried) and reads the next two sources while it works on two.  What it gives
// depends on the launch.  With few groups, where a CU holds few waves: 1.43 ms
// with the compiler's loop, 1.07 with this one, at 1914 groups (5e5 particles,
// items as below).  On a full chip the clock gives way instead (2.15 GHz with
// the compiler's loop): the 2^24 ring's launch 78.0 -> 77.1 ms, 64 Plummer
// spheres 1.79 -> 1.78.  The two sources' chains interleaved instruction by
// instruction were no faster alone and 2% slower there (78.2 ms): the power
// limit again.
//
// Registers, mass in the loop: ax, ay, az v57 v59 v61; xi, yi, zi v49 v51 v53;
// eps2 v55; sources v32-35, v36-39, v40-43, v44-47; temporaries v48, v50 and
// the odd ones up to v77.  Equal masses: ax, ay, az v40 v46 v52; xi, yi, zi v41
// v47 v53; eps2 v59; sources v42-45, v48-51, v54-57, v60-63; temporaries v58
// and v64 to v71.  Address v79.  The loop reads two sources past the last one
// (the tile is padded by 16) and waits for them before it ends.
#define SUB(d, a, b) "v_sub_f32 v" #d ", v" #a ", v" #b "\n\t"
#define MUL(d, a, b) "v_mul_f32 v" #d ", v" #a ", v" #b "\n\t"
#define FMA(d, a, b, c) "v_fma_f32 v" #d ", v" #a ", v" #b ", v" #c "\n\t"
#define FMAC(d, a, b) "v_fmac_f32 v" #d ", v" #a ", v" #b "\n\t"
#define RSQ(d, a) "v_rsq_f32 v" #d ", v" #a "\n\t"
#define LDS4(a, b, addr, off) "ds_read_b128 v[" #a ":" #b "], v" #addr " offset:" #off "\n\t"
// one source (x, y, z, m) with temporaries; the s_nop keeps v_rsq_f32 and its first use two instructions apart
#define PAIR_MASS(x, y, z, m, dy, r, t, u, f)                                                                  \
    SUB(z, z, 53) SUB(dy, y, 51) SUB(x, x, 49) FMA(r, z, z, 55) FMA(t, dy, dy, r) FMA(u, x, x, t) RSQ(r, u)    \
    "s_nop 0\n\t" MUL(t, r, r) MUL(u, m, r) MUL(f, u, t) FMAC(57, f, x) FMAC(59, f, dy) FMAC(61, f, z)
#define PAIR_EQM(x, y, z, r, t, f, u)                                                                          \
    SUB(z, z, 53) SUB(y, y, 47) SUB(x, x, 41) FMA(r, z, z, 59) FMA(t, y, y, r) FMA(u, x, x, t) RSQ(r, u)       \
    "s_nop 0\n\t" MUL(t, r, r) MUL(f, r, t) FMAC(40, f, x) FMAC(46, f, y) FMAC(52, f, z)
// two, the second on other temporaries
#define PAIR2_MASS(x, y, z, m, X, Y, Z, M)                                                                     \
    PAIR_MASS(x, y, z, m, 48, 63, 67, 75, 71) PAIR_MASS(X, Y, Z, M, 50, 65, 69, 77, 73)
#define PAIR2_EQM(x, y, z, X, Y, Z) PAIR_EQM(x, y, z, 58, 67, 69, 66) PAIR_EQM(X, Y, Z, 65, 64, 71, 68)

template <bool EQM>
__device__ __forceinline__ void pair_loop(uint32_t addr, int n4, float xi, float yi, float zi, float eps2, float &ax,
                                          float &ay, float &az) {
    if constexpr (EQM) {
        asm volatile(LDS4(42, 45, 79, 0) LDS4(48, 51, 79, 16)
                     ".p2align 6\n"
                     "Lpair%=:\n\t"
                     LDS4(54, 57, 79, 32) LDS4(60, 63, 79, 48)
                     "s_waitcnt lgkmcnt(2)\n\t"
                     PAIR2_EQM(42, 43, 44, 48, 49, 50)
                     "v_add_u32 v79, 64, v79\n\t"
                     LDS4(42, 45, 79, 0) LDS4(48, 51, 79, 16)
                     "s_waitcnt lgkmcnt(2)\n\t"
                     PAIR2_EQM(54, 55, 56, 60, 61, 62)
                     "s_sub_u32 %[n], %[n], 1\n\t"
                     "s_cmp_lg_u32 %[n], 0\n\t"
                     "s_cbranch_scc1 Lpair%=\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "+{v40}"(ax), "+{v46}"(ay), "+{v52}"(az), "+{v79}"(addr), [n] "+s"(n4)
                     : "{v41}"(xi), "{v47}"(yi), "{v53}"(zi), "{v59}"(eps2)
                     : "memory", "scc", "v42", "v43", "v44", "v45", "v48", "v49", "v50", "v51", "v54", "v55", "v56",
                       "v57", "v58", "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v71");
    } else {
        asm volatile(LDS4(32, 35, 79, 0) LDS4(36, 39, 79, 16)
                     ".p2align 6\n"
                     "Lpair%=:\n\t"
                     LDS4(40, 43, 79, 32) LDS4(44, 47, 79, 48)
                     "s_waitcnt lgkmcnt(2)\n\t"
                     PAIR2_MASS(32, 33, 34, 35, 36, 37, 38, 39)
                     "v_add_u32 v79, 64, v79\n\t"
                     LDS4(32, 35, 79, 0) LDS4(36, 39, 79, 16)
                     "s_waitcnt lgkmcnt(2)\n\t"
                     PAIR2_MASS(40, 41, 42, 43, 44, 45, 46, 47)
                     "s_sub_u32 %[n], %[n], 1\n\t"
                     "s_cmp_lg_u32 %[n], 0\n\t"
                     "s_cbranch_scc1 Lpair%=\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "+{v57}"(ax), "+{v59}"(ay), "+{v61}"(az), "+{v79}"(addr), [n] "+s"(n4)
                     : "{v49}"(xi), "{v51}"(yi), "{v53}"(zi), "{v55}"(eps2)
                     : "memory", "scc", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42",
                       "v43", "v44", "v45", "v46", "v47", "v48", "v50", "v63", "v65", "v67", "v69", "v71", "v73",
                       "v75", "v77");
    }
}
#undef SUB
#undef MUL
#undef FMA
#undef FMAC
#undef RSQ
#undef LDS4
#undef PAIR_MASS
#undef PAIR_EQM
#undef PAIR2_MASS
#undef PAIR2_EQM

// byte address of an LDS object
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

// whether a pass has the hand-scheduled loop
template <typename R, bool POT, bool ZERO_EPS, bool CLAMP>
constexpr bool PAIR_LOOP = sizeof(R) == 4 && !POT && !ZERO_EPS && !CLAMP;
// unrolling of the C++ loops: they take the last one to three sources after pair_loop
template <bool TAIL_ONLY>
constexpr int UNROLL = TAIL_ONLY ? 1 : 8;

// One pass of a wave over sources [j0, j1) of the LDS tile.  The bounds are
// the same for every lane of the wave; taking them through readfirstlane
// keeps the loop control on the scalar unit, so the vector unit issues only
// the pair arithmetic (every lane reads the same LDS entry: a broadcast).
// CLAMP (particle sources with the collision branch on): r^2 + eps^2 is
// raised to at least rce2 = rc^2 + eps^2 and its smallest value kept in cmin.
// EQM (particle sources of an equal-mass system): the common mass is taken
// out of the loop and applied to the sums at the end.
template <typename R, bool POT, bool ZERO_EPS, bool CLAMP, bool EQM>
__device__ __forceinline__ void interact(const typename V4<R>::T *tile, int j0, int j1, R xi, R yi, R zi, R eps2,
                                         R rce2, R &ax, R &ay, R &az, R &pot, R &cmin) {
    j0 = __builtin_amdgcn_readfirstlane(j0);
    j1 = __builtin_amdgcn_readfirstlane(j1);
#pragma unroll 8
    for (int j = j0; j < j1; ++j) {
        const typename V4<R>::T s = tile[j];
        const R dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
        R r2 = fma_r<R>(dx, dx, fma_r<R>(dy, dy, fma_r<R>(dz, dz, eps2)));
        if (CLAMP) {
            cmin = fmin(cmin, r2);
            r2 = fmax(r2, rce2);
        }
        R ri = rsqrt_r<R>(r2);
        if (ZERO_EPS && !CLAMP) ri = (r2 > (R)0) ? ri : (R)0;
        const R mri = EQM ? ri : s.w * ri;
        const R f = mri * (ri * ri);
        ax = fma_r<R>(f, dx, ax);
        ay = fma_r<R>(f, dy, ay);
        az = fma_r<R>(f, dz, az);
        if (POT) pot -= mri;
    }
}

// The same pass when the lanes of a wave work on different source ranges
// (sub-slices of a small group): lane base jb, common length L.
template <typename R, bool POT, bool ZERO_EPS, bool CLAMP, bool EQM>
__device__ __forceinline__ void interact_lanes(const typename V4<R>::T *tile, int jb, int L, R xi, R yi, R zi,
                                               R eps2, R rce2, R &ax, R &ay, R &az, R &pot, R &cmin) {
    L = __builtin_amdgcn_readfirstlane(L);
    const typename V4<R>::T *t = tile + jb;
    int k0 = 0;
    if constexpr (PAIR_LOOP<R, POT, ZERO_EPS, CLAMP>) {
        const int n4 = L >> 2;
        if (n4 > 0) pair_loop<EQM>(lds_address(t), n4, xi, yi, zi, eps2, ax, ay, az);
        k0 = max(n4, 0) * 4;
    }
#pragma unroll UNROLL<PAIR_LOOP<R, POT, ZERO_EPS, CLAMP>>
    for (int k = k0; k < L; ++k) {
        const typename V4<R>::T s = t[k];
        const R dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
        R r2 = fma_r<R>(dx, dx, fma_r<R>(dy, dy, fma_r<R>(dz, dz, eps2)));
        if (CLAMP) {
            cmin = fmin(cmin, r2);
            r2 = fmax(r2, rce2);
        }
        R ri = rsqrt_r<R>(r2);
        if (ZERO_EPS && !CLAMP) ri = (r2 > (R)0) ? ri : (R)0;
        const R mri = EQM ? ri : s.w * ri;
        const R f = mri * (ri * ri);
        ax = fma_r<R>(f, dx, ax);
        ay = fma_r<R>(f, dy, ay);
        az = fma_r<R>(f, dz, az);
        if (POT) pot -= mri;
    }
}

// One lane's pass over tile entries [jl0, jl0 + L): the whole wave on one
// range (sub == 1) or each sub-slice on its own.
template <typename R, bool POT, bool ZERO_EPS, bool CLAMP, bool EQM>
__device__ __forceinline__ void tile_pass(const typename V4<R>::T *tile, int sub, int jl0, int L, R xi, R yi, R zi,
                                          R eps2, R rce2, R &ax, R &ay, R &az, R &pot, R &cmin) {
    if (!PAIR_LOOP<R, POT, ZERO_EPS, CLAMP> && sub == 1)
        interact<R, POT, ZERO_EPS, CLAMP, EQM>(tile, jl0, jl0 + L, xi, yi, zi, eps2, rce2, ax, ay, az, pot, cmin);
    else
        interact_lanes<R, POT, ZERO_EPS, CLAMP, EQM>(tile, jl0, L, xi, yi, zi, eps2, rce2, ax, ay, az, pot, cmin);
}

// Contact terms of Eq. (2) for the pair (i, j), both sorted indices, in
// FP64 from the absolute positions and velocities: the decision
// dx*dx + dy*dy + dz*dz <= rc^2, then spring, dashpot and the potential of the
// gravity part inside the contact sphere, added to the thread's FP64 sums
// c[0], c[FT], c[2 FT], c[3 FT] (x, y, z, potential) in LDS.  Values are
// loaded only as far as the decision needs them: contacts are rare.
template <bool POT>
__device__ __forceinline__ void contact_term(uint32_t i, uint32_t j, const DevState &d, double *c) {
    const double4 p = d.pos[i];
    const double4 q = d.pos[j];
    const double ex = q.x - p.x, ey = q.y - p.y, ez = q.z - p.z;
    const double d2 = ex * ex + ey * ey + ez * ez;
    const double rc2 = d.rc * d.rc;
    if (d2 == 0.0) {
        // i itself (or a coincident particle): no term at all; take back the
        // potential the pair loop added at the clamped distance
        if (POT) c[3 * FT] += d.G * q.w / sqrt(rc2 + d.eps2);
        return;
    }
    if (!(d2 <= rc2)) return;
    const double4 vi = d.vel[i];
    const double4 vj = d.vel[j];
    const double r = sqrt(d2);
    const double rv = ex * (vj.x - vi.x) + ey * (vj.y - vi.y) + ez * (vj.z - vi.z);
    const double fc = q.w / (p.w + q.w) * (d.kappa * (r - d.rc) / r + d.eta * rv / d2);
    c[0 * FT] += fc * ex;
    c[1 * FT] += fc * ey;
    c[2 * FT] += fc * ez;
    if (POT) {
        const double rce2 = rc2 + d.eps2;
        c[3 * FT] -= d.G * q.w * ((rc2 - d2) / (2.0 * rce2 * sqrt(rce2)));
    }
}

// The contact candidates of one lane's particle i among tile entries
// [jb, jb + L): entries whose FP32 squared distance (the pair loop's own
// expression) is within rcd2, a bound that rounding of the relative
// coordinates cannot cross.  jidx holds the sorted index of each entry.
// A term costs two dependent rounds of global loads, and the lanes' candidates
// lie at different entries: taken one by one they were serial, and each
// particle is a candidate of its own (64 rounds per chunk).  So i itself needs
// no loads, the others are noted and taken side by side, in the lane's own
// order, and entries are looked at eight together, so that their LDS reads
// overlap.  130003 particles in 841 groups: 0.198 -> 0.137 ms per evaluation
// (0.093 without this pass); 2^22 in 54436 groups: 3.71 -> 3.26 ms.
template <typename R, bool POT>
__device__ __forceinline__ void contact_pass(const typename V4<R>::T *tile, const uint32_t *jidx, int jb, int L,
                                             R xi, R yi, R zi, R eps2, R rcd2, bool on, uint32_t i,
                                             const DevState &d, double *c) {
    if (!on) return;
    uint64_t noted = 0;          // up to four entries, 16 bits each, the first one lowest
    int n = 0;
    auto take = [&] {
        for (; n > 0; --n, noted >>= 16) contact_term<POT>(i, jidx[jb + (int)(noted & 0xffff)], d, c);
    };
    auto r2_of = [&](int k) {
        const typename V4<R>::T s = tile[jb + k];
        const R dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
        return fma_r<R>(dx, dx, fma_r<R>(dy, dy, fma_r<R>(dz, dz, eps2)));
    };
    auto note = [&](int k) {
        if (r2_of(k) <= rcd2) {
            if (jidx[jb + k] == i) {
                if (POT) contact_term<POT>(i, i, d, c);
            } else {
                noted |= (uint64_t)k << (16 * n);
                if (++n == 4) take();
            }
        }
    };
    int k = 0;
    for (; k + 8 <= L; k += 8) {
        R m = r2_of(k);
#pragma unroll
        for (int u = 1; u < 8; ++u) m = fmin(m, r2_of(k + u));
        if (m <= rcd2)
#pragma unroll 1
            for (int u = 0; u < 8; ++u) note(k + u);
    }
#pragma unroll 1
    for (; k < L; ++k) note(k);
    take();
}

// Work items of the persistent blocks: an item is 256 particles of a group (or
// what it has), so a group's particles are summed alike however many groups a
// launch has.  Items come in descending cost and Morton order: a block starts
// with the item of its number and goes on from one counter, so that blocks in
// flight work on neighbouring groups, whose sources stay in L2.  (Half of the
// items dealt to the blocks in turn, without the counter, took the 2^24 ring's
// launch from 77 to 105 ms: the blocks drift apart.)  Whole groups as items left
// the chip waiting for the last large ones when groups are few: 1.78 -> 1.43 ms
// at 1914 groups of up to 512.  The counter serves one pop per 12 ns, which is
// why the first items need none and empty ones do not exist (0.396 -> 0.364 ms at
// 16077 groups of the 2^20 ring, 77.1 -> 75.9 at 2^24, with the pop beside the
// results' writes).  A pop before the last sums, or a whole item ahead, gave
// nothing or bound the item to a block that was late (1.27 ms at 1914 groups).

// A work item's record in scalar registers: one load, a word per lane.  Read
// as a struct it went to vector registers (the kernel writes memory, so the
// compiler takes no scalar loads).
__device__ __forceinline__ ForceItem uniform_item(const ForceItem *p) {
    constexpr int W = sizeof(ForceItem) / 4;
    static_assert(W <= 64, "one word per lane");
    const int lane = __lane_id();
    const uint32_t v = reinterpret_cast<const uint32_t *>(p)[lane < W ? lane : 0];
    union {
        ForceItem item;
        uint32_t word[W];
    } u;
#pragma unroll
    for (int k = 0; k < W; ++k) u.word[k] = __builtin_amdgcn_readlane(v, k);
    return u.item;
}

// Workgroups per CU: the kernels' register caps, and what a launch starts, so
// that every block is resident from the start (a block's first item is the one
// of its number, among the most expensive; a block that waits for room would
// begin it when the others have emptied the queue).
// FP32: 6 (24 waves); the pair loop needs them to hide LDS and rsqrt latency
// (measured: 100 VGPRs / 4 waves per SIMD ran 18% slower; the collision
// variant, at 5 without spills, ran 3% slower than at 6 with some 40 spilled;
// in the gravity-only one pair_loop's named registers push 29 out, saved around
// the tiles: 0.6 of the 1.8 GB that a launch on 2^24 particles writes).
// FP64 gravity-only: 5 (<= 96 VGPRs, no spills); with the collision branch 3
// (141 VGPRs; uncapped, the variant with potentials took 169 and held 2 of the
// 3: 130003 particles in 3084 groups 0.178 -> 0.128 ms per evaluation, 2^20 in
// 3039 groups 1.92 -> 1.47 ms).
template <typename R, bool COLL>
struct ForceOcc {
    static constexpr int blocks = sizeof(R) == 4 ? 6 : (COLL ? 3 : 5);
};

template <typename R, bool POT, bool ZERO_EPS, bool COLL, int TJ>
// kick_h != 0: also apply the closing half kick v += kick_h a of a
// leapfrog step to each particle, as a separate pass over v and a would (the
// collision branch reads other particles' velocities, so it never fuses).
// TJ: sources per LDS tile (512, or 256 in the FP32 gravity-only kernels).
__global__ void __launch_bounds__(FT, (ForceOcc<R, COLL>::blocks)) k_force(DevState d, double kick_h) {
    static_assert(TJ == 256 || TJ == TJ_MAX, "tile of 256 or 512 sources");
    using T4 = typename V4<R>::T;
    // tail and eighths mode (below) in the FP32 kernels without the collision branch
    constexpr bool TAIL = sizeof(R) == 4 && !COLL;
    // FP32: sub-slices of 8, 16 or 32 lanes (below)
    constexpr bool POW2 = sizeof(R) == 4;
    constexpr int PAD = POW2 ? 16 : 64;
    __shared__ T4 tile[TJ + PAD];
    __shared__ uint32_t lbeg[LC];
    __shared__ uint32_t lscan[LC + 1];
    __shared__ R red[4][4][64];
    __shared__ uint32_t s_item;
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t jidx[COLL ? TJ : 1];            // sorted index of each particle-tile entry
    __shared__ double cacc[COLL ? 4 : 1][COLL ? FT : 1];  // per-thread FP64 contact sums
    // the particle ids of a leaf chunk, in list order, so that staging a
    // source is one LDS read instead of a search over the leaf offsets
    constexpr bool LIST_IDS = sizeof(R) == 4 && !COLL;
    __shared__ uint32_t pid[LIST_IDS ? PIDX : 1];

    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = __lane_id();
    const R eps2 = (R)d.eps2;
    const R rce2 = (R)(d.rc * d.rc + d.eps2);
    // detection margin: a bound on how far FP32 (FP64) rounding of the
    // group-relative coordinates can move a squared distance
    constexpr double U = sizeof(R) == 4 ? 0x1p-20 : 0x1p-49;

    const uint32_t items = __builtin_amdgcn_readfirstlane(d.cnt->n_items);
    // the item is the same for the whole workgroup: keep it (and all values
    // derived from it) in scalar registers
    for (uint32_t item = blockIdx.x; item < items;) {
        const ForceItem gi = uniform_item(d.force_items + item);
        const double4 cen = make_double4(gi.cx, gi.cy, gi.cz, 0.0);
        // FP32: an equal-mass system's particles enter the pair loop with unit
        // mass, node masses in units of that mass, the sums scaled at the end
        const double m0 = sizeof(R) == 4 ? gi.m0 : 0.0;
        const bool eqm = m0 > 0.0;
        const double gscale = eqm ? d.G * m0 : d.G;
        const double inv_m0 = eqm ? gi.inv_m0 : 1.0;
        const unsigned long long pc0 = gi.pc_off, pp0 = gi.pp_off;
        const uint32_t npc = gi.npc, npp = gi.npp;

        const uint32_t nb = gi.count;
        // Waves take 64-particle chunks of the block (n_ic of them), the
        // waves left over splitting the source range (split ways).  A chunk
        // of at most 32 particles -- a small group, or the last chunk of a
        // larger one -- spreads its wave over sub sub-slices of its source
        // range, cw lanes each.  FP32: 2, 4 or 8 of 32, 16 or 8 lanes (powers of
        // two, their divisions are shifts), with TAIL the sizes between in the
        // modes below.  FP64 (there tail and eighths mode hand sums over at twice
        // the cost: 0.335 -> 0.385 ms at 9311 groups of 21): as many as fit up to
        // 8, of exactly the chunk's particles: 3 for 17 to 21 instead of 2
        // (0.324 -> 0.298 ms at those groups).  With FP32 collisions that would
        // save 5% of the kernel and change its sums by their rounding.
        const int n_ic = (int)((nb + 63) >> 6);
        const int split_sh = n_ic == 1 ? 2 : (n_ic == 2 ? 1 : 0);
        const int split = 1 << split_sh;                         // 4 / n_ic
        const int ichunk = w % n_ic;
        const int jslice = w / n_ic;
        const bool wave_on = jslice < split;
        const int cnt_w = min(64, (int)nb - 64 * ichunk);
        // Slices of 8 particles in the chunk.  With 3, 5 or 7 of them the
        // chunk runs in eighths mode: lanes 0..8S-1 hold the particles and
        // take the first S eighths of the wave's source range; each of the
        // 8-S other groups of 8 lanes takes one of the last eighths for the
        // S slices in turn and hands each slice's partial sums to the lanes
        // that own them.  Every lane then runs S/8 of the range.
        const int s8 = (cnt_w + 7) >> 3;
        const bool e8 = TAIL && (s8 == 3 || s8 == 5 || s8 == 7);
        const int cw_sh = e8 ? 6 : (cnt_w <= 8 ? 3 : (cnt_w <= 16 ? 4 : (cnt_w <= 32 ? 5 : 6)));
        const int sub_sh = 6 - cw_sh;
        const int fit = 64 / max(cnt_w, 8);
        const int sub = POW2 ? 1 << sub_sh : fit;
        const int cw = POW2 ? 1 << cw_sh : (fit == 1 ? 64 : cnt_w);
        // lane / cw: exact, as 64 / 65536 is below 1 / cw
        const int part = POW2 ? lane >> cw_sh : lane * ((65536 + cw - 1) / cw) >> 16;
        // A chunk of 41 to 48 particles runs in tail mode: lanes 0..47 hold
        // the particles and take the first three quarters of the wave's
        // source range; lanes 48..63 take the last quarter for the three
        // 16-particle slices in turn and hand each slice's partial sums to
        // the lanes that own them.  Every lane then runs 3/4 of the range
        // instead of a full wave running all of it.
        const bool tailm = TAIL && cnt_w > 40 && cnt_w <= 48;
        const int last_cnt = (int)nb - 64 * (n_ic - 1);
        // the block's last chunk is sub-sliced, tailed or in eighths
        const bool any_sub = last_cnt <= (TAIL ? 56 : 32);
        const uint32_t il = 64 * ichunk + (lane - part * cw);
        const bool ion = wave_on && il < nb && (POW2 || part < sub);
        const uint32_t i = gi.begin + il;
        R xi = 0, yi = 0, zi = 0;
        if (ion) {
            const double4 p = d.pos[i];
            xi = (R)(p.x - cen.x);
            yi = (R)(p.y - cen.y);
            zi = (R)(p.z - cen.z);
        }
        R ax = 0, ay = 0, az = 0, pot = 0;
        R rcd2 = 0, cmin = 0;
        if (COLL) {
            const double n1 = fabs((double)xi) + fabs((double)yi) + fabs((double)zi);
            const double rcd = d.rc * (1.0 + U) + 0.5 * U * n1;
            rcd2 = (R)((rcd * rcd) * (1.0 + U) + d.eps2 * (1.0 + U));
#pragma unroll
            for (int a = 0; a < 4; ++a) cacc[a][tid] = 0.0;
        }

        // The staged tile holds cntt sources.  FP32: with a sub-sliced chunk in
        // the block the tile is padded with massless far sources to a multiple of
        // 8 split entries and cut at multiples of 8, so that every part has
        // the same length; full chunks still stop at the last real entry.
        // FP64: it is padded with 64 of them, each wave cuts it into split
        // sub parts of one length, an odd one when its lanes read several parts
        // at once (they then lie in different banks).
        // particles: whether the tile holds particle sources (the only ones
        // the collision branch applies to).
        auto compute_tile = [&](uint32_t cntt, bool particles) {
            const int ct = (int)cntt;
            const int cntp = !POW2 ? ct + PAD
                             : any_sub ? ((ct + (8 << split_sh) - 1) >> (3 + split_sh)) << (3 + split_sh)
                                       : ct;
            for (int t = ct + tid; t < cntp; t += FT) tile[t] = mk4<R>((R)1e18, (R)1e18, (R)1e18, (R)0);
            __syncthreads();
            if (wave_on) {
                // this lane's part of the range, [jl0, jl0 + L); the wave's, [jb, je)
                int jb = 0, je = 0, jl0, L;
                if constexpr (!POW2) {
                    const int parts = split * sub;
                    L = (ct + parts - 1) / parts;
                    if (sub == 1) {
                        jl0 = jslice * L;
                        L = max(0, min(L, ct - jl0));
                    } else {
                        L |= 1;
                        jl0 = (jslice * sub + min(part, sub - 1)) * L;
                    }
                } else {
                    if (any_sub) {
                        const int q = cntp >> 3;
                        jb = 8 * ((q * jslice) >> split_sh);
                        je = 8 * ((q * (jslice + 1)) >> split_sh);
                    } else {
                        jb = (ct * jslice) >> split_sh;
                        je = (ct * (jslice + 1)) >> split_sh;
                    }
                    if (sub == 1) {
                        jl0 = jb;
                        L = max(0, min(je, ct) - jb);
                    } else {
                        L = (je - jb) >> sub_sh;
                        jl0 = jb + part * L;
                    }
                }
                bool clamp = false;
                if constexpr (COLL) clamp = particles;
                const bool eq = particles && eqm;
                if (clamp) {
                    cmin = (R)1e30;
                    if (eq)
                        tile_pass<R, POT, ZERO_EPS, true, true>(tile, sub, jl0, L, xi, yi, zi, eps2, rce2, ax, ay,
                                                                az, pot, cmin);
                    else
                        tile_pass<R, POT, ZERO_EPS, true, false>(tile, sub, jl0, L, xi, yi, zi, eps2, rce2, ax,
                                                                 ay, az, pot, cmin);
                    // the real entries only: the padding has no particle, and at a radius of 1e18 it is in reach
                    if (__ballot(ion && cmin <= rcd2) != 0)
                        contact_pass<R, POT>(tile, jidx, jl0, min(L, ct - jl0), xi, yi, zi, eps2, rcd2, ion, i, d,
                                             &cacc[0][tid]);
                } else if (e8) {
                    const int Q = (je - jb) >> 3;
                    const int lg = lane >> 3;
                    const bool tail_lane = lg >= s8;
#pragma unroll 1
                    for (int pq = 0; pq < s8; ++pq) {
                        const int src = 8 * pq + (lane & 7);
                        const R tx = __shfl(xi, src, 64), ty = __shfl(yi, src, 64), tz = __shfl(zi, src, 64);
                        if (tail_lane) {
                            xi = tx;
                            yi = ty;
                            zi = tz;
                            ax = ay = az = pot = (R)0;
                        }
                        // owners: eighth pq of their own slice; others: their own eighth
                        const int j0 = jb + (tail_lane ? lg : pq) * Q;
                        if (eq)
                            interact_lanes<R, POT, ZERO_EPS, false, true>(tile, j0, Q, xi, yi, zi, eps2, rce2,
                                                                          ax, ay, az, pot, cmin);
                        else
                            interact_lanes<R, POT, ZERO_EPS, false, false>(tile, j0, Q, xi, yi, zi, eps2, rce2,
                                                                           ax, ay, az, pot, cmin);
                        for (int t = s8; t < 8; ++t) {
                            const int tl = 8 * t + (lane & 7);
                            const R sx = __shfl(ax, tl, 64), sy = __shfl(ay, tl, 64), sz = __shfl(az, tl, 64),
                                    sp = __shfl(pot, tl, 64);
                            if (lg == pq) {
                                ax += sx;
                                ay += sy;
                                az += sz;
                                pot += sp;
                            }
                        }
                    }
                } else if (tailm) {
                    const int Q = (je - jb) >> 2;
                    const bool tail_lane = lane >= 48;
#pragma unroll 1
                    for (int pq = 0; pq < 3; ++pq) {
                        const int src = 16 * pq + (lane & 15);
                        const R tx = __shfl(xi, src, 64), ty = __shfl(yi, src, 64), tz = __shfl(zi, src, 64);
                        if (tail_lane) {
                            xi = tx;
                            yi = ty;
                            zi = tz;
                            ax = ay = az = pot = (R)0;
                        }
                        const int j0 = tail_lane ? jb + 3 * Q : jb + pq * Q;
                        if (eq)
                            interact_lanes<R, POT, ZERO_EPS, false, true>(tile, j0, Q, xi, yi, zi, eps2, rce2,
                                                                          ax, ay, az, pot, cmin);
                        else
                            interact_lanes<R, POT, ZERO_EPS, false, false>(tile, j0, Q, xi, yi, zi, eps2, rce2,
                                                                           ax, ay, az, pot, cmin);
                        const int tl = 48 + (lane & 15);
                        const R sx = __shfl(ax, tl, 64), sy = __shfl(ay, tl, 64), sz = __shfl(az, tl, 64),
                                sp = __shfl(pot, tl, 64);
                        if ((lane >> 4) == pq) {
                            ax += sx;
                            ay += sy;
                            az += sz;
                            pot += sp;
                        }
                    }
                } else if (eq) {
                    tile_pass<R, POT, ZERO_EPS, false, true>(tile, sub, jl0, L, xi, yi, zi, eps2, rce2, ax, ay,
                                                             az, pot, cmin);
                } else {
                    tile_pass<R, POT, ZERO_EPS, false, false>(tile, sub, jl0, L, xi, yi, zi, eps2, rce2, ax, ay,
                                                              az, pot, cmin);
                }
            }
            __syncthreads();
        };

        // the first leaves of the particle list, loaded beside the first nodes
        uint32_t lb = 0, lc = 0;
        if ((uint32_t)tid < npp) {
            const uint32_t leaf = d.pp_pool[pp0 + tid];
            lb = d.nd_begin[leaf];
            lc = d.nd_count[leaf];
        }

        // ---- node list: centre of mass and mass of each accepted node
        for (uint32_t t0 = 0; t0 < npc; t0 += TJ) {
            const uint32_t cntt = min((uint32_t)TJ, npc - t0);
            for (uint32_t e = tid; e < cntt; e += FT) {
                const double4 m = d.nd_mom[d.pc_pool[pc0 + t0 + e]];
                tile[e] = mk4<R>((R)(m.x - cen.x), (R)(m.y - cen.y), (R)(m.z - cen.z), (R)(m.w * inv_m0));
            }
            compute_tile(cntt, false);
        }

        // ---- particle list: the particles of each listed leaf
        for (uint32_t l0 = 0; l0 < npp; l0 += LC) {
            const uint32_t nl = min((uint32_t)LC, npp - l0);
            if (l0 != 0) {
                lc = 0;
                if ((uint32_t)tid < nl) {
                    const uint32_t leaf = d.pp_pool[pp0 + l0 + tid];
                    lb = d.nd_begin[leaf];
                    lc = d.nd_count[leaf];
                }
            }
            // exclusive scan of leaf sizes over the workgroup
            const uint32_t inc = wave_incl_scan(lc);
            if (lane == 63) wsum[w] = inc;
            __syncthreads();
            uint32_t off = 0, tot = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                off += (k < w) ? wsum[k] : 0u;
                tot += wsum[k];
            }
            lbeg[tid] = lb;
            lscan[tid] = off + inc - lc;
            // a chunk of at most PIDX particles lists them all (each thread its
            // leaf's); a larger one (a few big level-21 leaves) searches
            const bool ids = LIST_IDS && tot <= (uint32_t)PIDX;
            if (ids)
                for (uint32_t k = 0; k < lc; ++k) pid[off + inc - lc + k] = lb + k;
            __syncthreads();
            for (uint32_t p0 = 0; p0 < tot; p0 += TJ) {
                const uint32_t cntt = min((uint32_t)TJ, tot - p0);
                for (uint32_t e = tid; e < cntt; e += FT) {
                    const uint32_t f = p0 + e;
                    uint32_t j;
                    if (ids) {
                        j = pid[f];
                    } else {
                        uint32_t lo = 0, hi = nl - 1;          // last k with lscan[k] <= f
                        while (lo < hi) {
                            const uint32_t mid = (lo + hi + 1) >> 1;
                            if (lscan[mid] <= f) lo = mid; else hi = mid - 1;
                        }
                        j = lbeg[lo] + (f - lscan[lo]);
                    }
                    const double4 q = d.pos[j];
                    tile[e] = mk4<R>((R)(q.x - cen.x), (R)(q.y - cen.y), (R)(q.z - cen.z), (R)q.w);
                    if (COLL) jidx[e] = j;
                }
                compute_tile(cntt, true);
            }
        }

        // ---- add the j-slices in a fixed order and write FP64 results
        if (POW2 && cw < 64) {
#pragma unroll
            for (int off = 32; off >= 8; off >>= 1) {
                if (off < cw) break;
                ax += __shfl_xor(ax, off, 64);
                ay += __shfl_xor(ay, off, 64);
                az += __shfl_xor(az, off, 64);
                pot += __shfl_xor(pot, off, 64);
            }
        }
        red[0][w][lane] = ax;
        red[1][w][lane] = ay;
        red[2][w][lane] = az;
        red[3][w][lane] = pot;
        __syncthreads();
        if (ion && jslice == 0 && lane < cw) {
            R sx = 0, sy = 0, sz = 0, sp = 0;
            for (int k = 0; k < split; ++k) {
                const int ww = k * n_ic + ichunk;
                for (int l = lane; l < (POW2 ? lane + 1 : sub * cw); l += cw) {
                    sx += red[0][ww][l];
                    sy += red[1][ww][l];
                    sz += red[2][ww][l];
                    sp += red[3][ww][l];
                }
            }
            double gx = gscale * (double)sx, gy = gscale * (double)sy, gz = gscale * (double)sz;
            if (d.amag) d.amag[i] = sqrt(gx * gx + gy * gy + gz * gz);
            if (d.central_mass != 0.0) {
                const double4 p = d.pos[i];
                const double r2 = p.x * p.x + p.y * p.y + p.z * p.z;
                const double r = sqrt(r2);
                const double f = -d.G * d.central_mass / (r2 * r);
                gx += f * p.x;
                gy += f * p.y;
                gz += f * p.z;
            }
            double gp = POT ? gscale * (double)sp : 0.0;
            if (COLL) {
                // contact sums of the threads that worked on particle i, in a fixed order
                double cx = 0, cy = 0, cz = 0, cp = 0;
                for (int k = 0; k < split; ++k)
                    for (int sb = 0; sb < sub; ++sb) {
                        const int th = (k * n_ic + ichunk) * 64 + sb * cw + lane;
                        cx += cacc[0][th];
                        cy += cacc[1][th];
                        cz += cacc[2][th];
                        cp += cacc[3][th];
                    }
                gx += cx;
                gy += cy;
                gz += cz;
                gp += cp;
            }
            d.acc[i] = make_double4(gx, gy, gz, POT ? gp : 0.0);
            if (!COLL && kick_h != 0.0) {
                double4 v = d.vel[i];
                v.x = v.x + kick_h * gx;
                v.y = v.y + kick_h * gy;
                v.z = v.z + kick_h * gz;
                d.vel[i] = v;
            }
        }
        // the next item, popped while the first wave writes its results; the
        // counter wraps to 0 with the launch's last pop (every item pops once)
        if (tid == FT - 1) s_item = atomicInc(&d.cnt->item_head, items - 1) + gridDim.x;
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(s_item);
    }
}

// n_cu compute units, items: an upper bound of the launch's items
template <typename R, bool POT, bool ZERO_EPS, bool COLL, int TJ>
void launch_kernel(const DevState &d, size_t items, int n_cu, double kick_h, hipStream_t s) {
    const unsigned blocks = (unsigned)std::min<size_t>((size_t)n_cu * ForceOcc<R, COLL>::blocks, items);
    k_force<R, POT, ZERO_EPS, COLL, TJ><<<blocks, FT, 0, s>>>(d, kick_h);
}

template <typename R, bool POT, bool ZERO_EPS>
void launch(const DevState &d, size_t items, int n_cu, double kick_h, hipStream_t s) {
    if (d.rc > 0.0) {
        launch_kernel<R, POT, ZERO_EPS, true, TJ_MAX>(d, items, n_cu, 0.0, s);
        return;
    }
    if constexpr (sizeof(R) == 4) {
        if (d.force_tile == 256) {
            launch_kernel<R, POT, ZERO_EPS, false, 256>(d, items, n_cu, kick_h, s);
            return;
        }
    }
    launch_kernel<R, POT, ZERO_EPS, false, TJ_MAX>(d, items, n_cu, kick_h, s);
}

template <typename R, bool POT>
void launch(const DevState &d, size_t items, int n_cu, double kick_h, hipStream_t s) {
    if (d.eps2 == 0.0) launch<R, POT, true>(d, items, n_cu, kick_h, s);
    else launch<R, POT, false>(d, items, n_cu, kick_h, s);
}

}  // namespace

namespace bhk {

void forces(const DevState &d, uint32_t n_groups, bool fp32, bool pot, int n_cu, double kick_h, hipStream_t s) {
    if (n_groups == 0) return;
    const size_t items = max_items(n_groups, d.n);
    if (fp32) {
        if (pot) launch<float, true>(d, items, n_cu, kick_h, s);
        else launch<float, false>(d, items, n_cu, kick_h, s);
    } else {
        if (pot) launch<double, true>(d, items, n_cu, kick_h, s);
        else launch<double, false>(d, items, n_cu, kick_h, s);
    }
}

}  // namespace bhk
