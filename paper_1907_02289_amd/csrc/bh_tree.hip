// bh_tree.hip -- tree construction, Iwasawa et al. (2019) Sec. 4.2 step (3a):
// root box and keys, sort and permutation, octree (all levels at once),
// monopole moments (Sec. 5.1: nodes act through their centre of mass),
// and the particle groups of step (3d) taken from the tree itself.
//
// Readings where the paper is silent:
//   root cube: lower corner at the per-axis minimum, side S the smallest
//     power of two strictly above the largest extent; grid coordinate
//     q = floor((x - lo) * 2^21 / S), at most 2^21 - 1; key = the 21 bits of
//     each axis interleaved, x the most significant bit of each triple.
//   tree: a node with more than n_leaf particles below level 21 is split
//     into its non-empty octants; nodes are numbered level by level.
//   groups: the first node on the way down from the root with at most
//     n_grp particles, or a leaf; ordered by first particle.
//
// Cylindrical tree coordinates (Sec. 4.3, Eq. (1)), when cyl_r > 0: for a
// narrow ring near radius cyl_r, cyl_r phi, r and z are locally Cartesian,
// so keys, cells and groups are built on (phi, r, z) while moments and
// forces stay Cartesian.  The root cell has side S = 2 pi cyl_r; its phi
// axis spans one turn, q = floor((phi + pi) 2^21 / (2 pi)); r and z use
// q = floor((v - min v) 2^21 / S).  phi comes from angle_of below, made of
// correctly rounded operations only, so the keys do not depend on a math
// library.
#include <algorithm>

#include "bh_internal.hpp"

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ int sys_of(const uint32_t *sys_off, int n_sys, uint32_t i) {
    int lo = 0, hi = n_sys - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (sys_off[mid] <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

inline unsigned grid_for(size_t n, size_t cap_blocks = 8192) {
    size_t b = (n + TPB - 1) / TPB;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return (unsigned)b;
}

// ---------------------------------------------------------------- cylindrical coordinates
constexpr double CYL_PI = 3.141592653589793;
constexpr double CYL_TAN_PI8 = 0.41421356237309503;   // tan(pi/8)

// arctan t for |t| <= tan(pi/8): the Maclaurin series t - t^3/3 + t^5/5 - ...
// (Abramowitz & Stegun 4.4.42) through t^29 (truncation below 2e-14),
// Horner's rule in t^2 from the top term down, coefficients (-1)^k / (2k+1).
__device__ __forceinline__ double atan_small(double t) {
    const double t2 = t * t;
    double p = 0.0;
#pragma unroll
    for (int k = 14; k >= 0; --k) {
        double c = 1.0 / (double)(2 * k + 1);
        if (k & 1) c = -c;
        p = p * t2 + c;
    }
    return t * p;
}

// Angle of (x, y) in [-pi, pi]: t = min/max(|x|, |y|) in [0, 1], reduced
// above tan(pi/8) by arctan t = pi/4 + arctan((t - 1)/(t + 1)) (A&S 4.4.34),
// then reflected into the octant and quadrant of (x, y); (0, 0) gives 0.
__device__ __forceinline__ double angle_of(double y, double x) {
    const double ax = fabs(x), ay = fabs(y);
    if (ax == 0.0 && ay == 0.0) return 0.0;
    const bool swap = ay > ax;
    const double t = swap ? ax / ay : ay / ax;
    double a = (t > CYL_TAN_PI8) ? 0.25 * CYL_PI + atan_small((t - 1.0) / (t + 1.0)) : atan_small(t);
    if (swap) a = 0.5 * CYL_PI - a;
    if (x < 0.0) a = CYL_PI - a;
    if (y < 0.0) a = -a;
    return a;
}

// The coordinates the tree is built on.
__device__ __forceinline__ void tree_coords(const DevState &d, double4 p, double c[3]) {
    if (d.cyl_r > 0.0) {
        c[0] = angle_of(p.y, p.x);
        c[1] = sqrt(p.x * p.x + p.y * p.y);
        c[2] = p.z;
    } else {
        c[0] = p.x;
        c[1] = p.y;
        c[2] = p.z;
    }
}

// ---------------------------------------------------------------- root box
// Blocks [first, end) of system s; one system alone has them all, without a load.
__device__ __forceinline__ void box_span(const DevState &d, int s, uint32_t &first, uint32_t &end) {
    first = d.n_sys == 1 ? 0u : d.box_off[s];
    end = d.n_sys == 1 ? d.box_blocks : d.box_off[s + 1];
}

// LOAD: from the caller's arrays, which the same pass copies into the library's
// records (a launch and 32 bytes per particle less than two passes).  Blocks are
// numbered over all systems, as many each as its own size asks for.
template <bool LOAD>
__global__ void __launch_bounds__(TPB) k_box_partial(DevState d) {
    const int s = sys_of(d.box_off, d.n_sys, blockIdx.x);
    const uint32_t b0 = d.sys_off[s], b1 = d.sys_off[s + 1];
    uint32_t first, end;
    box_span(d, s, first, end);
    // per axis 0..2 the tree coordinates, axis 3 the mass
    double lo[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, hi[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    bool bad = false;
    SysPtr sp;
    if (LOAD) sp = d.sys_tab[s];
    for (uint32_t i = b0 + (blockIdx.x - first) * TPB + threadIdx.x; i < b1; i += (end - first) * TPB) {
        double4 p;
        if (LOAD) {
            const uint32_t j = i - b0;
            p = make_double4(sp.x[j], sp.y[j], sp.z[j], sp.m[j]);
            d.pos_in[i] = p;
            d.vel_in[i] = sp.vx ? make_double4(sp.vx[j], sp.vy[j], sp.vz[j], 0.0) : make_double4(0.0, 0.0, 0.0, 0.0);
            d.idx_in[i] = i;
            if (d.amag_in) d.amag_in[i] = INFINITY;      // unknown until a force evaluation
        } else {
            p = d.pos_in[i];
        }
        bad |= !isfinite(p.x) || !isfinite(p.y) || !isfinite(p.z);
        double c[4];
        tree_coords(d, p, c);
        c[3] = p.w;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            lo[a] = fmin(lo[a], c[a]);
            hi[a] = fmax(hi[a], c[a]);
        }
    }
    if (bad) atomicOr(&d.cnt->flags[FLAG_NONFINITE], 1u);
    __shared__ double red[TPB / 64][8];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    const int w = threadIdx.x >> 6;
    if (__lane_id() == 0) {
        for (int a = 0; a < 4; ++a) {
            red[w][a] = lo[a];
            red[w][4 + a] = hi[a];
        }
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        int a = threadIdx.x;
        double v = red[0][a];
        for (int k = 1; k < TPB / 64; ++k) v = (a < 4) ? fmin(v, red[k][a]) : fmax(v, red[k][a]);
        d.box_part[(size_t)blockIdx.x * 8 + a] = v;
    }
}

__global__ void k_box_final(DevState d) {
    // one wave per system: lanes stride over the partials, then a wave reduction
    const int s = blockIdx.x;
    double lo[4], hi[4];
    for (int a = 0; a < 4; ++a) {
        lo[a] = INFINITY;
        hi[a] = -INFINITY;
    }
    uint32_t first, end;
    box_span(d, s, first, end);
    for (uint32_t b = first + threadIdx.x; b < end; b += 64) {
        const double *p = d.box_part + (size_t)b * 8;
        for (int a = 0; a < 4; ++a) {
            lo[a] = fmin(lo[a], p[a]);
            hi[a] = fmax(hi[a], p[4 + a]);
        }
    }
    for (int a = 0; a < 4; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    if (threadIdx.x != 0) return;
    // equal-mass systems let the force kernel take the common mass out of the pair loop
    d.sys_m0[s] = (lo[3] == hi[3] && lo[3] > 0.0) ? lo[3] : 0.0;
    if (d.cyl_r > 0.0) {
        // one turn of phi; r and z must fit the cell of side 2 pi cyl_r
        const double S = (2.0 * CYL_PI) * d.cyl_r;
        if (hi[1] - lo[1] >= S || hi[2] - lo[2] >= S) atomicOr(&d.cnt->flags[FLAG_EXTENT], 1u);
        d.box[s] = make_double4(-CYL_PI, lo[1], lo[2], 2097152.0 / S);
        return;
    }
    double w = 0.0;
    for (int a = 0; a < 3; ++a) {
        double e = hi[a] - lo[a];
        if (e > w) w = e;
    }
    int e2 = 0;
    if (w > 0.0) frexp(w, &e2);            // w < 2^e2 <= 2 w: S = 2^e2
    d.box[s] = make_double4(lo[0], lo[1], lo[2], ldexp(1.0, BH_MAXLEVEL - e2));
}

// ---------------------------------------------------------------- keys
__global__ void k_keys(DevState d, uint64_t *key, uint32_t *val) {
    uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < d.n; i += stride) {
        int s = sys_of(d.sys_off, d.n_sys, i);
        double4 b = d.box[s];
        double4 p = d.pos_in[i];
        double c[3], l[3] = {b.x, b.y, b.z};
        tree_coords(d, p, c);
        // the phi axis of cylindrical coordinates spans one turn
        const double k0 = d.cyl_r > 0.0 ? 2097152.0 / (2.0 * CYL_PI) : b.w;
        uint32_t q[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double t = (c[a] - l[a]) * (a == 0 ? k0 : b.w);
            double f = floor(t);
            q[a] = (f >= 2097151.0) ? 2097151u : (uint32_t)f;
        }
        key[i] = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
        val[i] = i;
    }
}

// Flags of the build and the counters of the walk that follows it.
__global__ void k_reset_flags(DevState d) {
    if (threadIdx.x < FLAG_COUNT) d.cnt->flags[threadIdx.x] = 0;
    if (threadIdx.x == 0) reset_walk_counters(d);
}

// ---------------------------------------------------------------- permute
__global__ void k_permute(DevState d) {
    uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < d.n; j += stride) {
        uint32_t src = d.val[j];
        d.pos[j] = d.pos_in[src];
        d.vel[j] = d.vel_in[src];
        const uint32_t gi = d.idx_in[src];
        d.idx[j] = gi;
        d.inv[gi] = j;
        if (d.amag && d.amag_in) d.amag[j] = d.amag_in[src];
        d.gmark[j] = 0;
    }
}

// ---------------------------------------------------------------- octree
// All levels at once from the sorted keys.  With cp(i, j) the number of
// leading octal digits that keys i and j share, a cell of level l starts at
// particle i when cp(i - 1, i) < l (or i starts its system); it is a node when
// its parent holds more than n_leaf particles, and it is split itself when
// cp(i, i + n_leaf) >= l.  So the nodes that start at particle i are those of
// levels first..last with
//   first = cp(i - 1, i) + 1, present only when the level first - 1 cell around
//           i holds more than n_leaf particles (its start is looked for among
//           the n_leaf particles before i),
//   last  = max(first, min(21, cp(i, i + n_leaf) + 1)).
// Ids run by (level, particle), so three launches do: nodes per level and tile
// of TREE_TILE particles, a scan of each level's tiles, and the nodes
// themselves, whose ranks inside a tile come from ballots.  (Level after
// level, 21 times count, three scans and emit, was 105 launches of 2.5 to
// 35 us: 320 us at 4096 particles, 660 at 2^20, 1500 at 2^24; the four launches
// now take 25, 60 and 690 us.)
// A block keeps its tile's keys, and TREE_PAD more on either side, in LDS: the
// searches around a particle are chains of dependent reads, and all but those
// of cells wider than the pad stay there.  One row of 64 particles per wave: a
// tile of 1024 (four rows in turn) takes 38 us instead of 15 at 4096
// particles, 51 instead of 41 at 2^20 and 514 instead of 445 at 2^24.
constexpr int TREE_TILE = TPB;
constexpr int TREE_ROWS = TREE_TILE / 64;
constexpr int TREE_PAD = 64;

struct TileKeys {
    const uint64_t *glob, *lds;
    uint32_t lo, hi;                            // particles [lo, hi) are in LDS
    __device__ __forceinline__ uint64_t operator[](uint32_t j) const {
        return j - lo < hi - lo ? lds[j - lo] : glob[j];
    }
};

__device__ __forceinline__ TileKeys tile_keys(const DevState &d, uint64_t *lds) {
    TileKeys t;
    const uint32_t i0 = blockIdx.x * TREE_TILE;
    t.glob = d.key;
    t.lds = lds;
    t.lo = i0 > TREE_PAD ? i0 - TREE_PAD : 0u;
    t.hi = min(d.n, i0 + TREE_TILE + TREE_PAD + 1);
    for (uint32_t j = t.lo + threadIdx.x; j < t.hi; j += TPB) lds[j - t.lo] = d.key[j];
    __syncthreads();
    return t;
}

// leading octal digits shared by two keys (0..21)
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x ? (__clzll((long long)x) - 1) / 3 : BH_MAXLEVEL;
}

// Levels first..last of the nodes that start at particle i of the system
// [b, e); none: first > last.
__device__ __forceinline__ void node_levels(const TileKeys &key, uint32_t i, uint32_t b, uint32_t e, uint32_t n_leaf,
                                            int &first, int &last) {
    const uint64_t k = key[i];
    int f = 0;
    first = BH_MAXLEVEL + 1;                       // none, unless found below
    last = 0;
    if (i > b) {
        const int L = common_digits(key[i - 1], k);
        if (L >= BH_MAXLEVEL) return;              // equal keys
        f = L + 1;
        const int sh = 3 * (BH_MAXLEVEL - L);      // L = 0: every key of the system
        // first particle of the parent's cell, at most n_leaf before i
        uint32_t lo = i - b > n_leaf ? i - n_leaf : b, hi = i;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (((key[mid] ^ k) >> sh) == 0) hi = mid; else lo = mid + 1;
        }
        if (e - lo <= n_leaf || ((key[lo + n_leaf] ^ k) >> sh) != 0) return;
    }
    int s = -1;
    if (e - i > n_leaf) s = common_digits(k, key[i + n_leaf]);
    first = f;
    last = max(f, min(BH_MAXLEVEL, s + 1));
}

// A particle's system and node levels.
struct TreeLevels {
    uint32_t i, b, e, sys;
    int first, last;
};
__device__ __forceinline__ TreeLevels tree_levels(const DevState &d, const TileKeys &key, uint32_t i) {
    TreeLevels t;
    t.i = i;
    t.first = BH_MAXLEVEL + 1;
    t.last = 0;
    t.b = t.e = t.sys = 0;
    if (t.i < d.n) {
        t.sys = (uint32_t)sys_of(d.sys_off, d.n_sys, t.i);
        t.b = d.sys_off[t.sys];
        t.e = d.sys_off[t.sys + 1];
        node_levels(key, t.i, t.b, t.e, (uint32_t)d.n_leaf, t.first, t.last);
    }
    return t;
}

__global__ void __launch_bounds__(TPB) k_tree_count(DevState d, uint32_t tiles) {
    __shared__ uint32_t cnt[BH_NLEVELS];
    __shared__ uint64_t lkey[TREE_TILE + 2 * TREE_PAD + 1];
    if (threadIdx.x < BH_NLEVELS) cnt[threadIdx.x] = 0;
    const TileKeys key = tile_keys(d, lkey);
    const TreeLevels t = tree_levels(d, key, blockIdx.x * TREE_TILE + threadIdx.x);
    const int lo = wave_min(t.first), hi = wave_max(t.last);
    for (int l = lo; l <= hi; ++l) {
        const uint64_t m = __ballot(l >= t.first && l <= t.last);
        if (m && __lane_id() == 0) atomicAdd(&cnt[l], (uint32_t)__popcll(m));
    }
    __syncthreads();
    if (threadIdx.x < BH_NLEVELS) d.tree_cnt[threadIdx.x * tiles + blockIdx.x] = cnt[threadIdx.x];
}

// One block per level: exclusive scan of the level's tile counts in place, and
// the level's total behind the last row.
__global__ void __launch_bounds__(1024) k_tree_scan(DevState d, uint32_t tiles) {
    __shared__ uint32_t wsum[16];
    uint32_t *row = d.tree_cnt + (size_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    const int w = threadIdx.x >> 6;
    for (uint32_t t0 = 0; t0 < tiles; t0 += 1024) {
        const uint32_t t = t0 + threadIdx.x;
        const uint32_t v = t < tiles ? row[t] : 0u;
        const uint32_t inc = wave_incl_scan(v);
        if (__lane_id() == 63) wsum[w] = inc;
        __syncthreads();
        uint32_t off = 0, tot = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            off += k < w ? wsum[k] : 0u;
            tot += wsum[k];
        }
        if (t < tiles) row[t] = carry + off + inc - v;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) d.tree_cnt[(size_t)BH_NLEVELS * tiles + blockIdx.x] = carry;
}

// End of the cell that starts at particle i, of the given digit shift, inside
// [i, e): called by whole waves (on = lanes with a cell).  Cells of up to 64
// particles: a binary search per lane; larger ones in turn, the 64 lanes
// probing the remaining range together.
__device__ __forceinline__ uint32_t cell_end(const TileKeys &key, bool on, uint32_t i, uint32_t e, int sh) {
    const uint64_t k = on ? key[i] >> sh : 0ull;
    uint32_t lo = i, hi = i;                      // key[lo] is in the cell, key[hi] is not (or hi = e)
    bool wide = false;
    if (on) {
        hi = e;
        if (e - i > 64) {
            wide = (key[i + 64] >> sh) == k;
            if (!wide) hi = i + 64;
        }
        if (!wide)
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if ((key[mid] >> sh) == k) lo = mid; else hi = mid;
            }
    }
    for (uint64_t m = __ballot(wide); m; m &= m - 1) {
        const int src = __ffsll((unsigned long long)m) - 1;
        const uint64_t ks = __shfl((unsigned long long)k, src, 64);
        const int shs = __shfl(sh, src, 64);
        uint32_t l = __shfl(i, src, 64) + 64, h = __shfl(e, src, 64);
        while (h - l > 1) {
            const uint32_t step = (h - l + 63) >> 6;
            const uint32_t p = l + (uint32_t)(__lane_id() + 1) * step;
            const bool in = p < h && p > l && (key.glob[p] >> shs) == ks;
            const uint32_t c = (uint32_t)__popcll(__ballot(in));
            l += c * step;
            h = h - l > step ? l + step : h;
        }
        if (__lane_id() == src) hi = h;
    }
    return hi;
}

// Up to this many tiles (16384 particles) a block adds up its level rows itself:
// some 2 us in place of the scan's launch and 3.
constexpr uint32_t TREE_FEW = 64;

__global__ void __launch_bounds__(TPB) k_tree_emit(DevState d, uint32_t tiles) {
    __shared__ uint64_t lkey[TREE_TILE + 2 * TREE_PAD + 1];
    __shared__ uint32_t rank[TREE_ROWS][BH_NLEVELS];   // nodes of a row, then its first id, per level
    static_assert(TREE_ROWS * BH_NLEVELS <= TPB && BH_NLEVELS < 64, "one thread per entry, one lane per level");
    // lanes 0..21 of the first wave: a level's total, first id and the tile's nodes before this one
    unsigned long long total = 0, end = 0;
    uint32_t before = 0;
    if (threadIdx.x < BH_NLEVELS) {
        const uint32_t *cnt = d.tree_cnt + (size_t)threadIdx.x * tiles;
        if (tiles <= TREE_FEW) {
            uint32_t all = 0;
#pragma unroll 8
            for (uint32_t t = 0; t < tiles; ++t) {
                const uint32_t c = cnt[t];
                before += t < blockIdx.x ? c : 0u;
                all += c;
            }
            total = all;
        } else {
            total = d.tree_cnt[(size_t)BH_NLEVELS * tiles + threadIdx.x];
            before = cnt[blockIdx.x];
        }
    }
    if (threadIdx.x < TREE_ROWS * BH_NLEVELS) (&rank[0][0])[threadIdx.x] = 0;
    const TileKeys key = tile_keys(d, lkey);
    const uint32_t row = threadIdx.x >> 6;
    const TreeLevels t = tree_levels(d, key, blockIdx.x * TREE_TILE + threadIdx.x);
    const int lo = wave_min(t.first), hi = wave_max(t.last);
    for (int l = lo; l <= hi; ++l) {
        const uint64_t m = __ballot(l >= t.first && l <= t.last);
        if (__lane_id() == 0) rank[row][l] = (uint32_t)__popcll(m);
    }
    if (row == 0) end = wave_incl_scan(total);
    __syncthreads();
    if (threadIdx.x < BH_NLEVELS) {
        uint32_t a = (uint32_t)min(end - total, (unsigned long long)d.node_cap) + before;
        for (int r = 0; r < TREE_ROWS; ++r) {
            const uint32_t c = rank[r][threadIdx.x];
            rank[r][threadIdx.x] = a;
            a += c;
        }
        if (blockIdx.x == 0) {
            const uint32_t e = (uint32_t)min(end, (unsigned long long)d.node_cap);
            d.cnt->lvl_off[threadIdx.x + 1] = e;
            if (threadIdx.x == 0) d.cnt->lvl_off[0] = 0;
            const uint64_t some = __ballot(total != 0);
            if (threadIdx.x == BH_NLEVELS - 1) {
                d.cnt->lvl_off[BH_NLEVELS + 1] = e;
                d.cnt->flags[FLAG_NODE_OVF] = end > d.node_cap ? 1u : 0u;
                d.cnt->max_level = 63 - __clzll((long long)some);
                d.cnt->n_groups = 0;
            }
        }
    }
    __syncthreads();
    uint32_t parent = 0;                        // this particle's node of the level above
    for (int l = lo; l <= hi; ++l) {
        const bool on = l >= t.first && l <= t.last;
        const uint64_t m = __ballot(on);
        const int sh = 3 * (BH_MAXLEVEL - l);
        const uint32_t end_i = cell_end(key, on, t.i, t.e, sh);
        if (!on) continue;
        const uint32_t u = rank[row][l] + (uint32_t)__popcll(m & lanemask_lt());
        // a node's first child starts where the node starts
        if (l > t.first && parent < d.node_cap) d.nd_first[parent] = u;
        parent = u;
        if (u >= d.node_cap) continue;          // overflow, flagged above: ids below the cap stay valid
        d.nd_prefix[u] = key[t.i] >> sh;
        d.nd_begin[u] = t.i;
        d.nd_count[u] = end_i - t.i;
        d.nd_meta[u] = make_meta(l, l < t.last ? 1u : 0u, 0, t.sys);    // the number of children follows
        if (l == t.last) d.nd_first[u] = 0;
    }
}

// Number of children and the walk's record of each node: the children are the
// nodes from the first child on that start inside the node.
__global__ void k_node_finalize(DevState d) {
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nn; v += stride) {
        const uint32_t meta = d.nd_meta[v];
        const uint32_t l = meta_level(meta);
        const uint64_t p = d.nd_prefix[v];
        uint32_t nch = 0, f = 0;
        if (meta_nch(meta)) {
            const uint32_t end = d.cnt->lvl_off[l + 2], e = d.nd_begin[v] + d.nd_count[v];
            f = d.nd_first[v];
            while (nch < 8 && f + nch < end && d.nd_begin[f + nch] < e) ++nch;
            d.nd_meta[v] = make_meta(l, nch, 0, meta_sys(meta));
        }
        const int sh = BH_MAXLEVEL - (int)l;
        const uint32_t cx = compact3(p >> 2) << sh, cy = compact3(p >> 1) << sh, cz = compact3(p) << sh;
        // a leaf has no first child: its record carries the particle count for the walk
        d.nd_walk[v] = make_int4((int)(cx | (l << 24)), (int)(cy | (nch << 24)), (int)cz,
                                 (int)(nch ? f : d.nd_count[v]));
    }
}

// ---------------------------------------------------------------- moments
// Bottom-up: a leaf sums its particles, an internal node its children (mass
// and mass-weighted centre).  All leaves of all levels in one launch, then the
// internal nodes level by level, and all top levels of at most MOM_TOP nodes
// in a single launch of one block with a
// barrier between levels.  One launch per level of the deepest possible tree
// was 22 launches of 2.4 to 31 us per refresh: 55 us at 4096 particles, 88 at
// 2^20; now 13 and 45 us.

// Adds n particles to the drift monitor's count of level l, for the lanes with
// on: one atomic per wave and level (lanes of a wave hold one level or two).
__device__ __forceinline__ void count_stale(const DevState &d, bool on, int l, uint32_t n) {
    for (uint64_t m = __ballot(on); m; m = __ballot(on)) {
        const int lv = __shfl(l, __ffsll((unsigned long long)m) - 1, 64);
        const bool mine = on && l == lv;
        const uint32_t sum = wave_sum(mine ? n : 0u);
        if (__lane_id() == 0) atomicAdd(&d.cnt->stale[lv], sum);
        on = on && !mine;
    }
}

__device__ __forceinline__ bool has_drifted(const DevState &d, double dr, uint32_t sys, int l) {
    const double side = ldexp((double)(1u << BH_MAXLEVEL) / d.box[sys].w, -l);
    return dr > d.drift_kappa * side;
}

// Mass and centre of mass of particles [b, e): eight in flight at once, summed in order.
__device__ __forceinline__ double4 leaf_sum(const DevState &d, uint32_t b, uint32_t e) {
    double M = 0, sx = 0, sy = 0, sz = 0;
    for (uint32_t i = b; i < e; i += 8) {
        double4 p[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k)
            if (i + k < e) p[k] = d.pos[i + k];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k)
            if (i + k < e) {
                M += p[k].w;
                sx += p[k].w * p[k].x;
                sy += p[k].w * p[k].y;
                sz += p[k].w * p[k].z;
            }
    }
    return make_double4(sx / M, sy / M, sz / M, M);
}

// Those of a node's children, in order.
__device__ __forceinline__ double4 child_sum(const double4 q[8], uint32_t nch) {
    double M = 0, sx = 0, sy = 0, sz = 0;
#pragma unroll
    for (uint32_t c = 0; c < 8; ++c)
        if (c < nch) {
            M += q[c].w;
            sx += q[c].w * q[c].x;
            sy += q[c].w * q[c].y;
            sz += q[c].w * q[c].z;
        }
    return make_double4(sx / M, sy / M, sz / M, M);
}

// Drift since the build: the largest distance by which a particle of
// the node has moved relative to the node's centre of mass,
//   leaf:     max_i |(x_i - x_i^b) - (c - c^b)|,
//   internal: max_k (drift_k + |(c_k - c_k^b) - (c - c^b)|),
// an upper bound of the leaf form over the node's particles.
__device__ __forceinline__ void leaf_moments(const DevState &d, uint32_t t0, uint32_t stride) {
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    const uint32_t end = (nn + 63u) & ~63u;          // whole waves: count_stale needs every lane
    for (uint32_t v = t0; v < end; v += stride) {
        const int4 wr = v < nn ? d.nd_walk[v] : make_int4(0, 1 << 24, 0, 0);
        const bool leaf = ((uint32_t)wr.y >> 24) == 0;
        const int l = (int)((uint32_t)wr.x >> 24);
        bool stale = false;
        if (leaf) {
            const uint32_t b = d.nd_begin[v], e = b + (uint32_t)wr.w;
            const double4 r = leaf_sum(d, b, e);
            d.nd_mom[v] = r;
            if (d.nd_drift) {
                const double4 rb = d.nd_mom_b[v];
                const double ux = r.x - rb.x, uy = r.y - rb.y, uz = r.z - rb.z;
                double dr = 0.0;
                for (uint32_t i = b; i < e; ++i) {
                    const double4 p = d.pos[i], q = d.pos_b[i];
                    const double ex = (p.x - q.x) - ux, ey = (p.y - q.y) - uy, ez = (p.z - q.z) - uz;
                    dr = fmax(dr, sqrt(ex * ex + ey * ey + ez * ez));
                }
                d.nd_drift[v] = dr;
                stale = has_drifted(d, dr, meta_sys(d.nd_meta[v]), l);
            }
            if (d.nd_quad) {
                double Q[6] = {0, 0, 0, 0, 0, 0};
                for (uint32_t i = b; i < e; ++i) {
                    double4 p = d.pos[i];
                    double dx = p.x - r.x, dy = p.y - r.y, dz = p.z - r.z;
                    Q[0] += p.w * dx * dx; Q[1] += p.w * dx * dy; Q[2] += p.w * dx * dz;
                    Q[3] += p.w * dy * dy; Q[4] += p.w * dy * dz; Q[5] += p.w * dz * dz;
                }
                double *o = d.nd_quad + (size_t)v * 6;
                for (int k = 0; k < 6; ++k) o[k] = Q[k];
            }
        }
        if (d.nd_drift) count_stale(d, stale, l, (uint32_t)wr.w);
    }
}

__global__ void __launch_bounds__(TPB) k_moments_leaf(DevState d) {
    leaf_moments(d, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// One internal node of level l; returns whether it has drifted.
__device__ __forceinline__ bool node_moments(const DevState &d, uint32_t v, int4 wr, int l) {
    const uint32_t nch = (uint32_t)wr.y >> 24, f = (uint32_t)wr.w;
    double4 q[8];
#pragma unroll
    for (uint32_t c = 0; c < 8; ++c)
        if (c < nch) q[c] = d.nd_mom[f + c];        // all in flight at once, summed in order
    const double4 r = child_sum(q, nch);
    d.nd_mom[v] = r;
    bool stale = false;
    if (d.nd_drift) {
        const double4 rb = d.nd_mom_b[v];
        const double ux = r.x - rb.x, uy = r.y - rb.y, uz = r.z - rb.z;
        double dr = 0.0;
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c)
            if (c < nch) {
                const double4 qb = d.nd_mom_b[f + c];
                const double ex = (q[c].x - qb.x) - ux, ey = (q[c].y - qb.y) - uy, ez = (q[c].z - qb.z) - uz;
                dr = fmax(dr, d.nd_drift[f + c] + sqrt(ex * ex + ey * ey + ez * ez));
            }
        d.nd_drift[v] = dr;
        stale = has_drifted(d, dr, meta_sys(d.nd_meta[v]), l);
    }
    if (d.nd_quad) {
        double Q[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c)
            if (c < nch) {
                const double *qc = d.nd_quad + (size_t)(f + c) * 6;
                double dx = q[c].x - r.x, dy = q[c].y - r.y, dz = q[c].z - r.z;
                Q[0] += qc[0] + q[c].w * dx * dx; Q[1] += qc[1] + q[c].w * dx * dy;
                Q[2] += qc[2] + q[c].w * dx * dz; Q[3] += qc[3] + q[c].w * dy * dy;
                Q[4] += qc[4] + q[c].w * dy * dz; Q[5] += qc[5] + q[c].w * dz * dz;
            }
        double *o = d.nd_quad + (size_t)v * 6;
        for (int k = 0; k < 6; ++k) o[k] = Q[k];
    }
    return stale;
}

// The internal nodes of level l, by the threads t0, t0 + stride, ...
__device__ __forceinline__ void level_moments(const DevState &d, int l, uint32_t t0, uint32_t stride) {
    const uint32_t v0 = d.cnt->lvl_off[l], v1 = d.cnt->lvl_off[l + 1];
    const uint32_t end = v0 + ((v1 - v0 + 63u) & ~63u);
    for (uint32_t v = v0 + t0; v < end; v += stride) {
        bool stale = false;
        if (v < v1) {
            const int4 wr = d.nd_walk[v];
            if (((uint32_t)wr.y >> 24) != 0) stale = node_moments(d, v, wr, l);
        }
        if (d.nd_drift) count_stale(d, stale, l, stale ? d.nd_count[v] : 0u);
    }
}

__global__ void __launch_bounds__(TPB) k_moments_level(DevState d, int l) {
    level_moments(d, l, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// Levels from `top` (or the deepest but one, whichever is higher up) to 0 in one block.
__global__ void __launch_bounds__(1024) k_moments_top(DevState d, int top) {
    for (int l = min(top, (int)d.cnt->max_level - 1); l >= 0; --l) {
        level_moments(d, l, threadIdx.x, 1024);
        __syncthreads();
    }
}

// A whole tree of at most MOM_SMALL nodes in one block, without drift and second
// moments: its nodes' records loaded at once, the moments passed from level to
// level in LDS.  Through memory a level waited 1.2 us for its children, and the
// leaves were a launch of their own: 4.5 + 10.3 us at 3001 particles, now 10.5,
// at 4096 4.7 + 11 and 13.
constexpr uint32_t MOM_SMALL = 4096;

__global__ void __launch_bounds__(1024) k_moments_small(DevState d) {
    __shared__ double4 mom[MOM_SMALL];
    constexpr int K = MOM_SMALL / 1024;
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    int4 wr[K];
    uint32_t begin[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t v = threadIdx.x + 1024 * k;
        wr[k] = v < nn ? d.nd_walk[v] : make_int4(0, 0, 0, 0);
        begin[k] = v < nn ? d.nd_begin[v] : 0u;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t v = threadIdx.x + 1024 * k;
        if (v < nn && ((uint32_t)wr[k].y >> 24) == 0) {
            const double4 r = leaf_sum(d, begin[k], begin[k] + (uint32_t)wr[k].w);
            mom[v] = r;
            d.nd_mom[v] = r;
        }
    }
    for (int l = (int)d.cnt->max_level - 1; l >= 0; --l) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t v = threadIdx.x + 1024 * k;
            const uint32_t nch = (uint32_t)wr[k].y >> 24, f = (uint32_t)wr[k].w;
            if (v < nn && nch != 0 && (int)((uint32_t)wr[k].x >> 24) == l) {
                double4 q[8];
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c)
                    if (c < nch) q[c] = mom[f + c];
                const double4 r = child_sum(q, nch);
                mom[v] = r;
                d.nd_mom[v] = r;
            }
        }
    }
}

// ---------------------------------------------------------------- groups
// Group flags for the current n_grp on an existing tree: a root is a group
// when small enough or a leaf; a child is a group when its parent is larger
// than n_grp and the child is small enough or a leaf (each node has exactly
// one parent, so the writes do not collide).  With packing, the flag marks
// the first node of each pack: the parent's thread walks its children in
// order and starts a new pack where the next small child no longer fits
// (the pack's particle count is taken later from the next group's start).
// Also marks the first particle of each group with the node's id plus one.
//
// Groups are numbered along the particles: marks per tile of particles, each
// tile's start as the sum of those before it, groups written and marks cleared
// tile by tile, then the boxes (and, with packing, the counts).  These four
// launches follow the tree's before its counters are read, so that one read
// serves both; a build that failed is left alone.  (With marks filled, three
// scan launches, the nodes' groups looked up and packed counts in a launch of
// their own it was 7 or 8, and a second read.)
__device__ __forceinline__ bool build_failed(const DevState &d) {
    return (d.cnt->flags[FLAG_NONFINITE] | d.cnt->flags[FLAG_EXTENT] | d.cnt->flags[FLAG_NODE_OVF]) != 0;
}

__global__ void k_regroup(DevState d) {
    if (build_failed(d)) return;
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    const uint32_t G = (uint32_t)d.n_grp;
    uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nn; v += stride) {
        const uint32_t meta = d.nd_meta[v], nch = meta_nch(meta), c = d.nd_count[v];
        if (v < (uint32_t)d.n_sys) {
            const bool grp = c <= G || nch == 0;
            d.nd_meta[v] = make_meta(meta_level(meta), nch, grp ? 1u : 0u, meta_sys(meta));
            if (grp) d.gmark[d.nd_begin[v]] = v + 1;
        }
        const uint32_t f = d.nd_first[v];
        uint32_t run = 0;    // particles in the open pack, 0 when none is open
        for (uint32_t k = 0; k < nch; ++k) {
            const uint32_t u = f + k;
            const uint32_t mu = d.nd_meta[u], cu = d.nd_count[u];
            bool grp = c > G && (cu <= G || meta_nch(mu) == 0);
            if (d.pack_groups && grp && cu <= G) {
                if (run > 0 && run + cu <= G) {
                    grp = false;             // joins the open pack
                    run += cu;
                } else {
                    run = cu;                // opens a pack
                }
            } else {
                run = 0;                     // a split child or an over-full leaf ends the run
            }
            if (grp != (meta_group(mu) != 0u))
                d.nd_meta[u] = make_meta(meta_level(mu), meta_nch(mu), grp ? 1u : 0u, meta_sys(mu));
            if (grp) d.gmark[d.nd_begin[u]] = u + 1;
        }
    }
}

// Particles per tile: at most 4096 tiles, whose counts a block adds up for itself.
uint32_t group_tile(uint32_t n) { return std::max(1024u, ((n + 4095) / 4096 + TPB - 1) / TPB * TPB); }

// d.tree_cnt, free once the octree is built, holds the tiles' counts.
__global__ void __launch_bounds__(TPB) k_group_count(DevState d, uint32_t tile) {
    __shared__ uint32_t red[TPB / 64];
    const uint32_t b = blockIdx.x * tile, e = min(b + tile, d.n);
    uint32_t c = 0;
    if (!build_failed(d))
        for (uint32_t i = b + threadIdx.x; i < e; i += TPB) c += d.gmark[i] != 0u;
    c = wave_sum(c);
    if (__lane_id() == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) d.tree_cnt[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void __launch_bounds__(TPB) k_group_emit(DevState d, uint32_t tile) {
    __shared__ uint32_t red[2][TPB / 64];
    if (build_failed(d)) return;
    const int w = threadIdx.x >> 6;
    uint32_t g = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += TPB) g += d.tree_cnt[t];
    g = wave_sum(g);
    if (__lane_id() == 0) red[0][w] = g;
    __syncthreads();
    g = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    __syncthreads();
    const uint32_t b = blockIdx.x * tile, e = min(b + tile, d.n);
    int r = 0;
    for (uint32_t i0 = b; i0 < e; i0 += TPB, r ^= 1) {
        const uint32_t i = i0 + threadIdx.x;
        const uint32_t mark = i < e ? d.gmark[i] : 0u;
        const uint64_t m = __ballot(mark != 0u);
        if (__lane_id() == 0) red[r][w] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t at = g + (uint32_t)__popcll(m & lanemask_lt());
        for (int k = 0; k < TPB / 64; ++k) {
            at += k < w ? red[r][k] : 0u;
            g += red[r][k];
        }
        if (mark) {
            const uint32_t v = mark - 1;
            d.grp[at] = GroupInfo{v, i, d.nd_count[v], meta_sys(d.nd_meta[v])};
            d.gmark[i] = 0;
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) d.cnt->n_groups = g;
}

// One wave per group: integer grid box from the keys, centre = midpoint of
// the FP64 bounding box of the group's particles.
__global__ void __launch_bounds__(TPB) k_group_box(DevState d) {
    const uint32_t ng = d.cnt->n_groups;
    const uint32_t wpb = TPB / 64;
    for (uint32_t g = blockIdx.x * wpb + (threadIdx.x >> 6); g < ng; g += gridDim.x * wpb) {
        GroupInfo gi = d.grp[g];
        if (d.pack_groups) {
            // the groups partition the sorted particles in order: a pack ends where the next group starts
            gi.count = (g + 1 < ng ? d.grp[g + 1].begin : (uint32_t)d.n) - gi.begin;
            if (__lane_id() == 0) d.grp[g].count = gi.count;
        }
        uint32_t qlo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, qhi[3] = {0, 0, 0};
        double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        for (uint32_t i = gi.begin + __lane_id(); i < gi.begin + gi.count; i += 64) {
            uint64_t k = d.key[i];
            uint32_t q[3] = {compact3(k >> 2), compact3(k >> 1), compact3(k)};
            double4 p = d.pos[i];
            double c[3] = {p.x, p.y, p.z};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                qlo[a] = min(qlo[a], q[a]);
                qhi[a] = max(qhi[a], q[a]);
                lo[a] = fmin(lo[a], c[a]);
                hi[a] = fmax(hi[a], c[a]);
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            qlo[a] = wave_min(qlo[a]);
            qhi[a] = wave_max(qhi[a]);
            lo[a] = wave_min(lo[a]);
            hi[a] = wave_max(hi[a]);
        }
        if (__lane_id() == 0) {
            d.g_lo[g] = make_int4((int)qlo[0], (int)qlo[1], (int)qlo[2], 0);
            d.g_hi[g] = make_int4((int)qhi[0] + 1, (int)qhi[1] + 1, (int)qhi[2] + 1, 0);
            d.g_cen[g] = make_double4(0.5 * (lo[0] + hi[0]), 0.5 * (lo[1] + hi[1]), 0.5 * (lo[2] + hi[2]), 0.0);
            if (d.g_rad) {
                const double ex = hi[0] - lo[0], ey = hi[1] - lo[1], ez = hi[2] - lo[2];
                d.g_rad[g] = 0.5 * sqrt(ex * ex + ey * ey + ez * ez);
            }
        }
        if (d.g_amin) d.g_amin[g] = group_budget(d, gi);
    }
}

}  // namespace

namespace bhk {

void root_box_keys(const DevState &d, bool load, hipStream_t s) {
    if (load) k_box_partial<true><<<d.box_blocks, TPB, 0, s>>>(d);
    else k_box_partial<false><<<d.box_blocks, TPB, 0, s>>>(d);
    k_box_final<<<d.n_sys, 64, 0, s>>>(d);
    if (sorts_small(d.n)) {
        k_keys<<<grid_for(d.n), TPB, 0, s>>>(d, d.key_tmp, d.val_tmp);
        sort_small(d.key_tmp, d.val_tmp, d.key, d.val, d.n, s, d.sys_off, d.n_sys);
    } else {
        k_keys<<<grid_for(d.n), TPB, 0, s>>>(d, d.key, d.val);
        radix_sort(d.key, d.val, d.key_tmp, d.val_tmp, d.n, 0, 63, d.hist, d.scan_tmp, s, d.sys_off, d.n_sys);
    }
}

void reset_flags(const DevState &d, hipStream_t s) {
    k_reset_flags<<<1, 64, 0, s>>>(d);
}

void permute(const DevState &d, hipStream_t s) {
    k_permute<<<grid_for(d.n), TPB, 0, s>>>(d);
}

uint32_t tree_tiles(uint32_t n) { return (n + TREE_TILE - 1) / TREE_TILE; }

size_t tree_cnt_words(uint32_t n) { return (size_t)BH_NLEVELS * (tree_tiles(n) + 1); }

void build_octree(const DevState &d, hipStream_t s) {
    const uint32_t tiles = tree_tiles(d.n);
    k_tree_count<<<tiles, TPB, 0, s>>>(d, tiles);
    if (tiles > TREE_FEW) k_tree_scan<<<BH_NLEVELS, 1024, 0, s>>>(d, tiles);
    k_tree_emit<<<tiles, TPB, 0, s>>>(d, tiles);
    k_node_finalize<<<grid_for(d.n, 4096), TPB, 0, s>>>(d);
}

// Levels of at most this many nodes share the single block of k_moments_top,
// one node per thread: 1.2 us per level.  At 4096 nodes the one CU's loads took
// 4 to 5 us per level, as much as a launch of its own.
constexpr uint32_t MOM_TOP = 1024;

void moment_plan(const uint32_t *lvl_off, uint32_t max_level, uint32_t n, int *deep, int *top, int *small) {
    // one block also sums the leaves: not when they hold many particles each
    *small = lvl_off[BH_NLEVELS] <= MOM_SMALL && n <= 4 * MOM_SMALL;
    int t = -1;
    while (t + 1 < (int)max_level && lvl_off[t + 2] - lvl_off[t + 1] <= MOM_TOP) ++t;
    // small trees: the one block takes every level, whatever the depth
    const bool all = t + 1 >= (int)max_level;
    *top = all ? BH_MAXLEVEL : t;
    *deep = all ? 0 : (int)max_level;
}

void moments(const DevState &d, hipStream_t s) {
    if (d.mom_small && !d.nd_drift && !d.nd_quad) {
        k_moments_small<<<1, 1024, 0, s>>>(d);
        return;
    }
    k_moments_leaf<<<grid_for(d.n, 4096), TPB, 0, s>>>(d);
    for (int l = d.mom_deep - 1; l > d.mom_top; --l) k_moments_level<<<grid_for(d.n / 4, 2048), TPB, 0, s>>>(d, l);
    if (d.mom_top >= 0) k_moments_top<<<1, 1024, 0, s>>>(d, d.mom_top);
}

__global__ void k_drift_snapshot(DevState d) {
    const uint32_t nn = d.cnt->lvl_off[BH_NLEVELS];
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t t0 = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t i = t0; i < d.n; i += stride) d.pos_b[i] = d.pos[i];
    for (uint32_t v = t0; v < nn; v += stride) d.nd_mom_b[v] = d.nd_mom[v];
    if (t0 < BH_NLEVELS) d.cnt->stale[t0] = 0;
}

__global__ void k_drift_clear(DevState d) {
    if (threadIdx.x < BH_NLEVELS) d.cnt->stale[threadIdx.x] = 0;
}

void drift_snapshot(const DevState &d, hipStream_t s) {
    k_drift_snapshot<<<grid_for(d.n, 4096), TPB, 0, s>>>(d);
}

void drift_clear(const DevState &d, hipStream_t s) {
    k_drift_clear<<<1, 64, 0, s>>>(d);
}

void make_groups(const DevState &d, hipStream_t s) {
    const uint32_t tile = group_tile(d.n), tiles = (d.n + tile - 1) / tile;
    k_regroup<<<grid_for(d.n, 4096), TPB, 0, s>>>(d);
    k_group_count<<<tiles, TPB, 0, s>>>(d, tile);
    k_group_emit<<<tiles, TPB, 0, s>>>(d, tile);
    k_group_box<<<grid_for((size_t)d.n * 64 / 8, 8192), TPB, 0, s>>>(d);
}

}  // namespace bhk
