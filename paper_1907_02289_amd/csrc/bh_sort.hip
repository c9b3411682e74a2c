// bh_sort.hip -- device-wide exclusive scan and stable sort of (key, value)
// pairs.
//
// The sort orders the particles' 63-bit keys for the tree build; the paper
// names sorting as the dominant cost of tree construction (Sec. 4.2) and
// uses a sample sort on its CPEs.  Three ways here, by size, all stable:
//   up to SMALL_MAX pairs: places counted by comparison over the whole chip;
//   up to SAMPLE_MAX: a sample sort.  Splitters from a sorted sample cut the
//     pairs into at most 1024 buckets of about 1000 to 2500, in one stable
//     scatter, and a block sorts each bucket in LDS: seven launches, and two
//     passes over memory instead of eight;
//   above: radix passes over memory with 8-bit
//     digits, per pass one histogram kernel, one scan of the (digit, block)
//     counts and one scatter kernel whose ranks come from wave-level digit
//     matching (eight ballots).  The scatter first orders its tile by digit in
//     LDS and then writes each digit's run to consecutive addresses.
// Below SAMPLE_MAX the radix passes are bound by their 40 launches (27 us a
// pass at 2^20 keys, 17 at 4096): 63-bit keys took 180 us of launches at 4096,
// 190 at 2e5, 270 at 2^20 and 330 at 2e6; now 10, 80, 100 and 185.
#include <type_traits>

#include "bh_internal.hpp"
#include "bh_sort_plan.hpp"

namespace {

using namespace bhk;

constexpr int SCAN_BLOCKS = 256;
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 4;

constexpr int RS_THREADS = 256;              // 4 waves
constexpr int RS_WAVE_ITEMS = 8;             // rounds of 64 keys per wave
constexpr int RS_TILE = RS_THREADS * RS_WAVE_ITEMS;   // 2048 keys per block

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *wsum, uint32_t *total) {
    // 256 threads = 4 waves; wsum: 4 words of LDS
    uint32_t inc = wave_incl_scan(v);
    int w = threadIdx.x >> 6;
    if (__lane_id() == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < SCAN_THREADS / 64; ++k) {
        uint32_t t = wsum[k];
        off += (k < w) ? t : 0u;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__global__ void __launch_bounds__(SCAN_THREADS) k_scan_reduce(const uint32_t *in, uint32_t n, uint32_t *part) {
    __shared__ uint32_t wsum[4];
    uint32_t chunk = (n + SCAN_BLOCKS - 1) / SCAN_BLOCKS;
    uint32_t b0 = blockIdx.x * chunk;
    uint32_t b1 = min(n, b0 + chunk);
    uint32_t s = 0;
    for (uint32_t i = b0 + threadIdx.x; i < b1; i += SCAN_THREADS) s += in[i];
    s = wave_sum(s);
    if (__lane_id() == 0) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// Every block adds up the partial sums before its own (a launch less than
// scanning them apart).
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_down(const uint32_t *in, uint32_t *out, uint32_t n,
                                                           const uint32_t *part) {
    static_assert(SCAN_BLOCKS == SCAN_THREADS, "one partial sum per thread");
    __shared__ uint32_t wsum[4];
    uint32_t chunk = (n + SCAN_BLOCKS - 1) / SCAN_BLOCKS;
    uint32_t b0 = blockIdx.x * chunk;
    uint32_t b1 = min(n, b0 + chunk);
    uint32_t carry;
    (void)block_excl_scan(threadIdx.x < blockIdx.x ? part[threadIdx.x] : 0u, wsum, &carry);
    for (uint32_t t0 = b0; t0 < b1; t0 += SCAN_THREADS * SCAN_ITEMS) {
        uint32_t v[SCAN_ITEMS];
        uint32_t base = t0 + threadIdx.x * SCAN_ITEMS;
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            v[k] = (base + k < b1) ? in[base + k] : 0u;
            s += v[k];
        }
        uint32_t tot;
        uint32_t ex = block_excl_scan(s, wsum, &tot) + carry;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            if (base + k < b1) out[base + k] = ex;
            ex += v[k];
        }
        carry += tot;
    }
}

__global__ void k_copy_pairs(const uint64_t *kin, const uint32_t *vin, uint64_t *kout, uint32_t *vout, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        kout[i] = kin[i];
        vout[i] = vin[i];
    }
}

// ---------------------------------------------------------------- radix sort
// Digit of element i: 8 key bits at `shift`, or (SYS) 8 bits of the system
// index that owns input index val[i] (sys_off: n_sys+1 ascending offsets).
template <bool SYS>
__device__ __forceinline__ uint32_t rs_digit(const uint64_t *key, const uint32_t *val, uint32_t i, int shift,
                                             const uint32_t *sys_off, int n_sys) {
    if (!SYS) return (uint32_t)(key[i] >> shift) & 255u;
    uint32_t v = val[i];
    int lo = 0, hi = n_sys - 1;          // last s with sys_off[s] <= v
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (sys_off[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return ((uint32_t)lo >> shift) & 255u;
}

template <bool SYS>
__global__ void __launch_bounds__(RS_THREADS) k_radix_hist(const uint64_t *key, const uint32_t *val, uint32_t n,
                                                          int shift, uint32_t *hist, uint32_t nb,
                                                          const uint32_t *sys_off, int n_sys) {
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    uint32_t base = blockIdx.x * RS_TILE;
#pragma unroll 4
    for (int r = 0; r < RS_WAVE_ITEMS; ++r) {
        uint32_t i = base + r * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&cnt[rs_digit<SYS>(key, val, i, shift, sys_off, n_sys)], 1u);
    }
    __syncthreads();
    hist[threadIdx.x * nb + blockIdx.x] = cnt[threadIdx.x];
}

template <bool SYS>
__global__ void __launch_bounds__(RS_THREADS) k_radix_scatter(const uint64_t *key_in, const uint32_t *val_in,
                                                             uint64_t *key_out, uint32_t *val_out,
                                                             uint32_t n, int shift,
                                                             const uint32_t *hist_scan, uint32_t nb,
                                                             const uint32_t *sys_off, int n_sys) {
    __shared__ uint32_t run[4][256];
    __shared__ uint32_t loc[256];                // block-local start of each digit's run
    __shared__ uint32_t gbase[256];              // global start of this block's run of each digit
    __shared__ uint32_t wsum[4];
    __shared__ uint64_t skey[RS_TILE];           // the tile in (digit, input) order
    __shared__ uint32_t sval[RS_TILE];
    __shared__ uint8_t sdig[RS_TILE];
    const int w = threadIdx.x >> 6;
    const int lane = __lane_id();
#pragma unroll
    for (int k = 0; k < 4; ++k) run[k][threadIdx.x] = 0;
    __syncthreads();

    const uint32_t base = blockIdx.x * RS_TILE + w * (RS_WAVE_ITEMS * 64);
    uint32_t digit[RS_WAVE_ITEMS];
    uint32_t rank[RS_WAVE_ITEMS];
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < RS_WAVE_ITEMS; ++r) {
        uint32_t i = base + r * 64 + lane;
        bool valid = i < n;
        uint32_t d = valid ? rs_digit<SYS>(key_in, val_in, i, shift, sys_off, n_sys) : 0u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t old = valid ? run[w][d] : 0u;
        __syncthreads();
        bool leader = valid && ((peers & lt) == 0);
        if (leader) run[w][d] = old + (uint32_t)__popcll(peers);
        __syncthreads();
        digit[r] = d;
        rank[r] = old + (uint32_t)__popcll(peers & lt);
    }
    // block-local start of each digit (scan over the digits), then of each
    // wave's share of it; the block's global start of each digit
    {
        const uint32_t t = threadIdx.x;
        const uint32_t c0 = run[0][t], c1 = run[1][t], c2 = run[2][t], c3 = run[3][t];
        uint32_t tot;
        const uint32_t ex = block_excl_scan(c0 + c1 + c2 + c3, wsum, &tot);
        loc[t] = ex;
        run[0][t] = ex;
        run[1][t] = ex + c0;
        run[2][t] = ex + c0 + c1;
        run[3][t] = ex + c0 + c1 + c2;
        gbase[t] = hist_scan[t * nb + blockIdx.x];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_WAVE_ITEMS; ++r) {
        const uint32_t i = base + r * 64 + lane;
        if (i < n) {
            const uint32_t lp = run[w][digit[r]] + rank[r];
            skey[lp] = key_in[i];
            sval[lp] = val_in[i];
            sdig[lp] = (uint8_t)digit[r];
        }
    }
    __syncthreads();
    // consecutive threads write consecutive slots of each digit's run
    const uint32_t t0 = blockIdx.x * RS_TILE;
    const uint32_t cnt = n - t0 < (uint32_t)RS_TILE ? n - t0 : (uint32_t)RS_TILE;
    for (uint32_t p = threadIdx.x; p < cnt; p += RS_THREADS) {
        const uint32_t d = sdig[p];
        const uint32_t pos = gbase[d] + (p - loc[d]);
        key_out[pos] = skey[p];
        val_out[pos] = sval[p];
    }
}

// ---------------------------------------------------------------- sort in one block
// system (of n_sys, offsets off) that owns input index v
__device__ __forceinline__ uint32_t owner(const uint32_t *off, int n_sys, uint32_t v) {
    int lo = 0, hi = n_sys - 1;          // last s with off[s] <= v
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return (uint32_t)lo;
}

// A block of T threads sorts up to CAP pairs by (system, key, index): a sample
// of SUB of them is ranked by counting and cuts the rest into SUB + 1 runs of
// about ten, and every pair counts the pairs of its run before it.  The index
// makes the order strict, so equal keys fall into many runs as well and the
// sort is stable.  Bound by the instructions of the comparisons: where the
// bucket's systems and keys span fewer than 51 bits (all but buckets across a
// top-level cell boundary) a pair is one 64-bit number, offset from the
// bucket's least pair above its index, and a comparison two instructions;
// elsewhere (WIDE) it takes the parts in turn.  Radix passes over digits in
// LDS took 80 instructions a pair and pass of 8 bits (2^20 keys in 1024
// buckets: 75 us with six passes; 31 this way).
template <int T, int CAP, bool SYS>
struct BlockSortLds {
    static constexpr int SUB = 128;
    uint64_t key[CAP];
    uint16_t idx[CAP], sys[SYS ? CAP : 1];
    uint64_t skey[SUB];                  // the sample in order
    uint16_t sidx[SUB], ssys[SYS ? SUB : 1];
    uint32_t start[SUB + 2], cnt[SUB + 1];
    unsigned long long agg[T / 64][3];
    uint32_t vr[2];
};

template <bool SYS>
__device__ __forceinline__ bool pair_less(uint32_t ya, uint64_t ka, uint32_t ia, uint32_t yb, uint64_t kb, uint32_t ib) {
    const bool l = ka < kb || (ka == kb && ia < ib);
    return SYS ? ya < yb || (ya == yb && l) : l;
}

// What a block's pairs span: key bits that differ, least and greatest key,
// first and last system.
struct PairSpan {
    unsigned long long diff, lo, hi;
    uint32_t sys0, sys1;
};

// WIDE: comparisons by (system, key, index); else key[] holds
// (key - span.lo) << 13 | index of one system.
template <int T, int E, bool SYS, bool WIDE, int CAP, bool LS>
__device__ __forceinline__ void block_sort(const uint64_t *kin, const uint32_t *vin, uint64_t *kout, uint32_t *vout,
                                           uint32_t cnt, const PairSpan &span, const uint32_t *sys_off, int n_sys,
                                           BlockSortLds<T, CAP, LS> &L) {
    using Lds = BlockSortLds<T, CAP, LS>;
    constexpr int SUB = Lds::SUB;
    static_assert(T >= 4 * SUB && (LS || !SYS) && CAP <= 8192 && (WIDE || !SYS), "");
    uint64_t k[E];
    uint32_t v[E], y[E], at[E];          // at: run << 16 | place in it
    auto less = [&](uint32_t ya, uint64_t ka, uint32_t ia, uint32_t yb, uint64_t kb, uint32_t ib) {
        if constexpr (WIDE) return pair_less<SYS>(ya, ka, ia, yb, kb, ib);
        else return ka < kb;
    };
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t q = r * T + threadIdx.x;
        k[r] = 0;
        v[r] = y[r] = 0;
        if (q < cnt) {
            k[r] = kin[q];
            if (!WIDE) k[r] = (k[r] - span.lo) << 13 | q;
            v[r] = vin[q];
            L.key[q] = k[r];
            if (SYS) {
                y[r] = owner(sys_off, n_sys, v[r]) - span.sys0;
                L.sys[q] = (uint16_t)y[r];
            }
        }
    }
    for (int t = threadIdx.x; t <= SUB; t += T) L.cnt[t] = 0;
    __syncthreads();
    // the sample: pair m cnt / sub for m < sub (SUB of them; fewer than SUB pairs: all), by fixed point
    const uint32_t sub = min((uint32_t)SUB, cnt);
    const uint32_t step = (cnt << 16) / sub;
    constexpr uint32_t R = T / SUB >= 8 ? 8 : 4;      // threads per sampled pair
    if (threadIdx.x < R * SUB) {
        const uint32_t m = threadIdx.x / R, p = threadIdx.x % R;
        const uint32_t i = m * step >> 16;
        uint32_t rank = 0, ys = 0;
        uint64_t ks = 0;
        if (m < sub) {
            ks = L.key[i];
            if (SYS) ys = L.sys[i];
#pragma unroll 8
            for (uint32_t j = p; j < sub; j += R) {
                const uint32_t jj = j * step >> 16;
                rank += less(SYS ? L.sys[jj] : 0u, L.key[jj], jj, ys, ks, i) ? 1u : 0u;
            }
        }
#pragma unroll
        for (uint32_t o = R / 2; o >= 1; o >>= 1) rank += __shfl_xor(rank, o, 64);
        if (p == 0) {
            const bool on = m < sub;            // slots past the sample: above every pair
            const uint32_t at_m = on ? rank : m;
            L.skey[at_m] = on ? ks : ~0ull;
            L.sidx[at_m] = (uint16_t)(on ? i : 0xffffu);
            if (SYS) L.ssys[at_m] = (uint16_t)(on ? ys : 0xffffu);
        }
    }
    __syncthreads();
    // sampled pairs not after this one: E searches side by side
    uint32_t lo[E];
    auto before = [&](int r, uint32_t m) {
        return less(y[r], k[r], r * T + threadIdx.x, SYS ? L.ssys[m] : 0u, L.skey[m], WIDE ? L.sidx[m] : 0u);
    };
#pragma unroll
    for (int r = 0; r < E; ++r) lo[r] = 0;
#pragma unroll
    for (uint32_t st = SUB / 2; st >= 1; st >>= 1)
#pragma unroll
        for (int r = 0; r < E; ++r)
            if (!before(r, lo[r] + st - 1)) lo[r] += st;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (!before(r, lo[r])) lo[r] += 1;
        at[r] = r * T + threadIdx.x < cnt ? lo[r] << 16 | atomicAdd(&L.cnt[lo[r]], 1u) : 0u;
    }
    __syncthreads();
    constexpr int PL = (SUB + 2 + 63) / 64;        // starts of the runs: PL counts per lane of a wave
    if (threadIdx.x < 64) {
        uint32_t c[PL], sum = 0;
#pragma unroll
        for (int j = 0; j < PL; ++j) {
            const int t = PL * threadIdx.x + j;
            c[j] = t <= SUB ? L.cnt[t] : 0u;
            sum += c[j];
        }
        uint32_t a = wave_incl_scan(sum) - sum;
#pragma unroll
        for (int j = 0; j < PL; ++j) {
            const int t = PL * threadIdx.x + j;
            if (t <= SUB + 1) L.start[t] = a;
            a += c[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t q = r * T + threadIdx.x;
        if (q < cnt) {
            const uint32_t p = L.start[at[r] >> 16] + (at[r] & 0xffffu);
            L.key[p] = k[r];
            if (WIDE) L.idx[p] = (uint16_t)q;
            if (SYS) L.sys[p] = (uint16_t)y[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t q = r * T + threadIdx.x;
        if (q < cnt) {
            const uint32_t b = L.start[at[r] >> 16], e = L.start[(at[r] >> 16) + 1];
            uint32_t pos = b;
            for (uint32_t p = b; p < e; p += 4) {           // four at a time: their reads overlap
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t w = min(p + u, e - 1);
                    const bool l = less(SYS ? L.sys[w] : 0u, L.key[w], WIDE ? L.idx[w] : 0u, y[r], k[r], q);
                    pos += l && p + u < e ? 1u : 0u;
                }
            }
            kout[pos] = WIDE ? k[r] : (k[r] >> 13) + span.lo;
            vout[pos] = v[r];
        }
    }
}

template <int T, int CAP, bool LS>
__device__ __forceinline__ PairSpan block_span(const uint64_t *kin, const uint32_t *vin, uint32_t cnt,
                                               const uint32_t *sys_off, int n_sys, BlockSortLds<T, CAP, LS> &L) {
    unsigned long long any = 0, lo = ~0ull, hi = 0;
    const unsigned long long first = kin[0];
    uint32_t vlo = 0xffffffffu, vhi = 0;
    for (uint32_t q = threadIdx.x; q < cnt; q += T) {
        const unsigned long long k = kin[q];
        any |= k ^ first;
        lo = k < lo ? k : lo;
        hi = k > hi ? k : hi;
        if (LS) {
            vlo = min(vlo, vin[q]);
            vhi = max(vhi, vin[q]);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) any |= __shfl_xor(any, o, 64);
    lo = wave_min(lo);
    hi = wave_max(hi);
    const int w = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        L.vr[0] = 0xffffffffu;
        L.vr[1] = 0;
    }
    if (__lane_id() == 0) {
        L.agg[w][0] = any;
        L.agg[w][1] = lo;
        L.agg[w][2] = hi;
    }
    __syncthreads();
    PairSpan s{0, ~0ull, 0, 0, 0};
    for (int q = 0; q < T / 64; ++q) {
        s.diff |= L.agg[q][0];
        s.lo = L.agg[q][1] < s.lo ? L.agg[q][1] : s.lo;
        s.hi = L.agg[q][2] > s.hi ? L.agg[q][2] : s.hi;
    }
    if (LS) {
        vlo = wave_min(vlo);
        vhi = wave_max(vhi);
        if (__lane_id() == 0) {
            atomicMin(&L.vr[0], vlo);
            atomicMax(&L.vr[1], vhi);
        }
        __syncthreads();
        s.sys0 = owner(sys_off, n_sys, L.vr[0]);
        s.sys1 = owner(sys_off, n_sys, L.vr[1]);
    }
    return s;
}

// Up to SMALL_MAX pairs: every pair's place counted over the whole chip in one
// launch, n^2 comparisons dealt to blocks of RANK_ROWS pairs (4096 pairs:
// 10 us; one block sorting them in its LDS took 36 to 43).  The
// sample sort ranks its sample the same way.
constexpr uint32_t RANK_ROWS = 32, RANK_CHUNK = 2048, RANK_THREADS = 1024;

// Ranks of pairs row0 .. row0 + 31 of the block among m pairs with systems
// sys(j): left in out[32] (LDS), ties by index.
template <bool SYS, typename F>
__device__ __forceinline__ void rank_rows(const uint64_t *key, F sys, uint32_t m, uint32_t *out) {
    __shared__ uint64_t sk[RANK_CHUNK];
    __shared__ uint32_t sy[SYS ? RANK_CHUNK : 1];
    // 8 groups of two waves, four rows each; the 128 threads of a group deal the pairs among them
    const uint32_t row0 = blockIdx.x * RANK_ROWS + 4 * (threadIdx.x >> 7), p = threadIdx.x & 127;
    uint64_t k[4];
    uint32_t y[4], rank[4] = {0, 0, 0, 0};
    if (threadIdx.x < RANK_ROWS) out[threadIdx.x] = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t i = min(row0 + r, m - 1);
        k[r] = key[i];
        y[r] = SYS ? sys(i) : 0u;
    }
    for (uint32_t c = 0; c < m; c += RANK_CHUNK) {
        const uint32_t len = min(RANK_CHUNK, m - c);
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < RANK_CHUNK / RANK_THREADS; ++u) {
            const uint32_t j = u * RANK_THREADS + threadIdx.x;
            if (j < len) {
                sk[j] = key[c + j];
                if (SYS) sy[j] = sys(c + j);
            }
        }
        __syncthreads();
        // equal pairs rank by index: counted in chunks before the rows', not in chunks after them
        auto count = [&](auto less) {
#pragma unroll 4
            for (uint32_t j = p; j < len; j += 128) {
                const uint64_t kj = sk[j];
                const uint32_t yj = SYS ? sy[j] : 0u;
#pragma unroll
                for (int r = 0; r < 4; ++r) rank[r] += less(yj, kj, c + j, r) ? 1u : 0u;
            }
        };
        if (c + len <= row0)
            count([&](uint32_t yj, uint64_t kj, uint32_t, int r) { return SYS ? yj < y[r] || (yj == y[r] && kj <= k[r]) : kj <= k[r]; });
        else if (c >= row0 + 4)
            count([&](uint32_t yj, uint64_t kj, uint32_t, int r) { return SYS ? yj < y[r] || (yj == y[r] && kj < k[r]) : kj < k[r]; });
        else
            count([&](uint32_t yj, uint64_t kj, uint32_t j, int r) { return pair_less<SYS>(yj, kj, j, y[r], k[r], row0 + r); });
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t s = wave_sum(rank[r]);
        if (__lane_id() == 0) atomicAdd(&out[4 * (threadIdx.x >> 7) + r], s);
    }
    __syncthreads();
}

template <bool SYS>
__global__ void __launch_bounds__(RANK_THREADS) k_sort_small(const uint64_t *key, const uint32_t *val, uint64_t *kout,
                                                            uint32_t *vout, uint32_t n, const uint32_t *sys_off,
                                                            int n_sys) {
    __shared__ uint32_t rank[RANK_ROWS];
    rank_rows<SYS>(key, [&](uint32_t j) { return owner(sys_off, n_sys, val[j]); }, n, rank);
    const uint32_t i = blockIdx.x * RANK_ROWS + threadIdx.x;
    if (threadIdx.x < RANK_ROWS && i < n) {
        kout[rank[threadIdx.x]] = key[i];
        vout[rank[threadIdx.x]] = val[i];
    }
}

// ---------------------------------------------------------------- sample sort
// n pairs, B buckets (8..1024) of n / B pairs on average, cut by a sample of 8 to
// 16 pairs per bucket (sample_plan).  A bucket outgrows the LDS of its block only
// where the sample happens to miss a stretch of its pairs (the plan states how
// often) or in an input made to defeat it; such a bucket is sorted by its block
// over memory.  Keys that fill a bucket by
// themselves show as repeated splitters and get a bucket of their own, which
// needs no sorting: with lb (ub) splitters below (not above)
// a pair, its bucket is ub, and lb + 1 when it equals two splitters or more.
constexpr int SS_THREADS = 512;                 // histogram and scatter
constexpr int SS_SORT = 512;                    // bucket sort: 1024 threads took 25 instead of 30 us at 2e5 pairs, 44 instead of 31 at 2^20
constexpr uint32_t SS_TILE = 4096;              // pairs per scatter block

struct SampleLayout {
    uint32_t buckets, per, tiles;               // buckets, samples per bucket, scatter tiles
    uint64_t stretch;                           // input pairs per sampled one, 32.32 fixed point
    uint64_t *split_key;                        // [BUCKETS_MAX]
    uint32_t *split_sys;                        // [BUCKETS_MAX]
    uint32_t *hist;                             // [buckets][tiles]
    uint16_t *bucket;                           // [n]
};

inline size_t ss_words(uint32_t n) {
    return 3 * (size_t)BUCKETS_MAX + (size_t)sample_plan(n, false).buckets * ((n + SS_TILE - 1) / SS_TILE) + (n + 1) / 2;
}

inline SampleLayout ss_layout(uint32_t n, const SamplePlan &p, uint32_t *scratch) {
    SampleLayout s;
    s.buckets = p.buckets;
    s.per = p.per;
    s.stretch = ((uint64_t)n << 32) / (s.buckets * s.per);
    s.tiles = (n + SS_TILE - 1) / SS_TILE;
    s.split_key = reinterpret_cast<uint64_t *>(scratch);
    s.split_sys = scratch + 2 * BUCKETS_MAX;
    s.hist = s.split_sys + BUCKETS_MAX;
    s.bucket = reinterpret_cast<uint16_t *>(s.hist + (size_t)s.buckets * s.tiles);
    return s;
}

// The sample: pair j of buckets * per comes from the j-th of as many equal
// stretches of the input, at a place that a hash of j picks; gathered into
// (ks, ys).
__global__ void k_ss_gather(const uint64_t *key, const uint32_t *val, const uint32_t *sys_off, int n_sys,
                            SampleLayout s, uint64_t *ks, uint32_t *ys) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= s.buckets * s.per) return;
    const uint32_t a = (uint32_t)((j * s.stretch) >> 32), b = (uint32_t)(((j + 1) * s.stretch) >> 32);
    const uint32_t h = (j + 1) * 2654435761u;
    const uint32_t i = a + (uint32_t)((uint64_t)(b - a) * h >> 32);
    ks[j] = key[i];
    ys[j] = n_sys > 1 ? owner(sys_off, n_sys, val[i]) : 0u;
}

// Splitters: every per-th of the sample by rank.
template <bool SYS>
__global__ void __launch_bounds__(RANK_THREADS) k_ss_rank(const uint64_t *ks, const uint32_t *ys, SampleLayout s) {
    __shared__ uint32_t rank[RANK_ROWS];
    const uint32_t m = s.buckets * s.per;
    rank_rows<SYS>(ks, [&](uint32_t j) { return ys[j]; }, m, rank);
    const uint32_t i = blockIdx.x * RANK_ROWS + threadIdx.x;
    if (threadIdx.x < RANK_ROWS && i < m) {
        const uint32_t r = rank[threadIdx.x];
        if (r > 0 && r % s.per == 0) {
            s.split_key[r / s.per - 1] = ks[i];
            s.split_sys[r / s.per - 1] = SYS ? ys[i] : 0u;
        }
    }
}

__global__ void __launch_bounds__(SS_THREADS) k_ss_hist(const uint64_t *key, const uint32_t *val, uint32_t n,
                                                       const uint32_t *sys_off, int n_sys, SampleLayout s) {
    __shared__ uint64_t sk[BUCKETS_MAX];
    __shared__ uint32_t ss[BUCKETS_MAX], cnt[BUCKETS_MAX];
    const uint32_t nsp = s.buckets - 1;
    for (uint32_t b = threadIdx.x; b < s.buckets; b += SS_THREADS) {
        cnt[b] = 0;
        if (b < nsp) {
            sk[b] = s.split_key[b];
            ss[b] = s.split_sys[b];
        }
    }
    __syncthreads();
    for (uint32_t i = blockIdx.x * SS_TILE + threadIdx.x; i < min(n, (blockIdx.x + 1) * SS_TILE); i += SS_THREADS) {
        const uint64_t k = key[i];
        const uint32_t y = n_sys > 1 ? owner(sys_off, n_sys, val[i]) : 0u;
        uint32_t lo = 0, hi = nsp;                  // splitters not above the pair
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (ss[mid] < y || (ss[mid] == y && sk[mid] <= k)) lo = mid + 1; else hi = mid;
        }
        if (lo >= 2 && sk[lo - 1] == k && ss[lo - 1] == y && sk[lo - 2] == k && ss[lo - 2] == y) {
            uint32_t a = 0, b = lo - 1;             // first splitter equal to the pair
            while (a < b) {
                const uint32_t mid = (a + b) >> 1;
                if (ss[mid] < y || (ss[mid] == y && sk[mid] < k)) a = mid + 1; else b = mid;
            }
            lo = a + 1;
        }
        s.bucket[i] = (uint16_t)lo;
        atomicAdd(&cnt[lo], 1u);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < s.buckets; b += SS_THREADS) s.hist[(size_t)b * s.tiles + blockIdx.x] = cnt[b];
}

__global__ void __launch_bounds__(SS_THREADS) k_ss_scatter(const uint64_t *key, const uint32_t *val, uint64_t *kout,
                                                          uint32_t *vout, uint32_t n, SampleLayout s) {
    constexpr int W = SS_THREADS / 64, E = SS_TILE / SS_THREADS;
    __shared__ uint16_t run[W][BUCKETS_MAX];
    const int w = threadIdx.x >> 6, lane = __lane_id();
    uint32_t *z = reinterpret_cast<uint32_t *>(&run[0][0]);
    for (uint32_t t = threadIdx.x; t < W * BUCKETS_MAX / 2; t += SS_THREADS) z[t] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * SS_TILE + w * (64 * E) + lane;
    uint32_t dr[E];                                 // bucket | rank in the wave << 16
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t i = base + 64 * r;
        const bool valid = i < n;
        const uint32_t d = valid ? s.bucket[i] : 0u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 10; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t old = run[w][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) run[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
        dr[r] = d | ((old + below) << 16);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < s.buckets; b += SS_THREADS) {
        uint32_t a = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const uint32_t c = run[q][b];
            run[q][b] = (uint16_t)a;
            a += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t i = base + 64 * r;
        if (i < n) {
            const uint32_t d = dr[r] & 0xffffu;
            const uint32_t pos = s.hist[(size_t)d * s.tiles + blockIdx.x] + run[w][d] + (dr[r] >> 16);
            kout[pos] = key[i];
            vout[pos] = val[i];
        }
    }
}

// A bucket larger than LDS holds: radix passes of the one block over memory,
// 1024 pairs at a time, between the two copies; ends in (ka, va).  run: LDS,
// [waves][256]; head: [256]; wsum: [waves].
__device__ void block_sort_memory(uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb, uint32_t cnt,
                                  unsigned long long diff, uint32_t sys0, uint32_t sys1, const uint32_t *sys_off,
                                  int n_sys, uint32_t (*run)[256], uint32_t *head, uint32_t *wsum) {
    constexpr int T = SS_SORT, W = T / 64;
    const int w = threadIdx.x >> 6, lane = __lane_id();
    uint64_t *ki = kb, *ko = ka;
    uint32_t *vi = vb, *vo = va;
    auto pass = [&](int sh, bool sys) {
        auto digit = [&](uint32_t q) -> uint32_t {
            return sys ? ((owner(sys_off, n_sys, vi[q]) - sys0) >> sh) & 255u : (uint32_t)(ki[q] >> sh) & 255u;
        };
        __syncthreads();
        for (int t = threadIdx.x; t < 256; t += T) head[t] = 0;
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < cnt; q += T) atomicAdd(&head[digit(q)], 1u);
        __syncthreads();
        uint32_t c = 0;
        if (threadIdx.x < 256) c = head[threadIdx.x];
        const uint32_t inc = wave_incl_scan(c);
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        if (threadIdx.x < 256) {
            uint32_t at = inc - c;
            for (int q = 0; q < w; ++q) at += wsum[q];
            head[threadIdx.x] = at;
        }
        for (uint32_t q0 = 0; q0 < cnt; q0 += T) {
            for (int t = threadIdx.x; t < W * 256; t += T) (&run[0][0])[t] = 0;
            __syncthreads();
            const uint32_t q = q0 + threadIdx.x;
            const bool valid = q < cnt;
            const uint32_t d = valid ? digit(q) : 0u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
            if (valid && below == 0) run[w][d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (valid) {
                uint32_t pos = head[d] + below;
                for (int p = 0; p < w; ++p) pos += run[p][d];
                ko[pos] = ki[q];
                vo[pos] = vi[q];
            }
            __syncthreads();
            if (threadIdx.x < 256) {
                uint32_t sum = 0;
                for (int p = 0; p < W; ++p) sum += run[p][threadIdx.x];
                head[threadIdx.x] += sum;
            }
            __syncthreads();
        }
        uint64_t *kt = ki; ki = ko; ko = kt;
        uint32_t *vt = vi; vi = vo; vo = vt;
    };
    for (int sh = 0; sh < 64; sh += 8)
        if ((diff >> sh) & 255u) pass(sh, false);
    for (int sh = 0; (sys1 - sys0) >> sh; sh += 8) pass(sh, true);
    __syncthreads();
    if (ki != ka)
        for (uint32_t q = threadIdx.x; q < cnt; q += T) {
            ka[q] = ki[q];
            va[q] = vi[q];
        }
}

// One block per bucket: from (kin, vin), where the scatter put it, to (kout, vout).
// Two blocks per CU, by LDS and by a cap of 128 VGPRs: without it three of the four
// instances took 129 to 153, room for one (2.2e6 pairs of 64 systems 0.63 -> 0.60 ms
// for keys, sort and permutation, 2.6e6 of one 0.79 -> 0.75).
template <int CAP, bool SYS>
__global__ void __launch_bounds__(SS_SORT, 4) k_ss_sort(uint64_t *kin, uint32_t *vin, uint64_t *kout, uint32_t *vout,
                                                       uint32_t n, const uint32_t *sys_off, int n_sys,
                                                       SampleLayout s) {
    __shared__ BlockSortLds<SS_SORT, CAP, SYS> L;
    constexpr int T = SS_SORT;
    const uint32_t b0 = s.hist[(size_t)blockIdx.x * s.tiles];
    const uint32_t b1 = blockIdx.x + 1 < s.buckets ? s.hist[(size_t)(blockIdx.x + 1) * s.tiles] : n;
    const uint32_t cnt = b1 - b0;
    if (cnt == 0) return;
    kin += b0;
    vin += b0;
    kout += b0;
    vout += b0;
    const PairSpan span = block_span(kin, vin, cnt, sys_off, n_sys, L);
    const bool one = span.sys0 == span.sys1;
    if (cnt > CAP) {
        if (span.diff == 0 && one) {
            for (uint32_t q = threadIdx.x; q < cnt; q += T) {
                kout[q] = kin[q];
                vout[q] = vin[q];
            }
        } else {
            // the pair arrays' LDS serves the passes' counters
            uint32_t(*run)[256] = reinterpret_cast<uint32_t(*)[256]>(L.key);
            block_sort_memory(kout, vout, kin, vin, cnt, span.diff, span.sys0, span.sys1, sys_off, n_sys, run,
                              reinterpret_cast<uint32_t *>(L.key) + (T / 64) * 256, L.cnt);
        }
        return;
    }
    auto sort = [&](auto sys, auto wide) {
        constexpr bool Y = decltype(sys)::value, WD = decltype(wide)::value;
        if (cnt <= T) block_sort<T, 1, Y, WD>(kin, vin, kout, vout, cnt, span, sys_off, n_sys, L);
        else if (cnt <= 2 * T) block_sort<T, 2, Y, WD>(kin, vin, kout, vout, cnt, span, sys_off, n_sys, L);
        else if (cnt <= 4 * T) block_sort<T, 4, Y, WD>(kin, vin, kout, vout, cnt, span, sys_off, n_sys, L);
        else if (cnt <= 8 * T) block_sort<T, 8, Y, WD>(kin, vin, kout, vout, cnt, span, sys_off, n_sys, L);
        else if constexpr (CAP > 8 * T) block_sort<T, 16, Y, WD>(kin, vin, kout, vout, cnt, span, sys_off, n_sys, L);
    };
    if (one && ((span.hi - span.lo) >> 51) == 0) {
        sort(std::false_type{}, std::false_type{});
        return;
    }
    if constexpr (SYS) {
        if (!one) {
            sort(std::true_type{}, std::true_type{});
            return;
        }
    }
    sort(std::false_type{}, std::true_type{});
}

}  // namespace

namespace bhk {

void scan_u32(const uint32_t *in, uint32_t *out, uint32_t n, uint32_t *tmp, hipStream_t s) {
    k_scan_reduce<<<SCAN_BLOCKS, SCAN_THREADS, 0, s>>>(in, n, tmp);
    k_scan_down<<<SCAN_BLOCKS, SCAN_THREADS, 0, s>>>(in, out, n, tmp);
}

size_t radix_hist_words(uint32_t n) {
    size_t nb = (n + RS_TILE - 1) / RS_TILE;
    if (nb == 0) nb = 1;
    const size_t sample = ss_words(n < SAMPLE_MAX ? n : SAMPLE_MAX);
    return nb * 256 > sample ? nb * 256 : sample;
}

bool sorts_small(uint32_t n) { return n <= SMALL_MAX; }

void sort_small(const uint64_t *key, const uint32_t *val, uint64_t *key_out, uint32_t *val_out, uint32_t n,
                hipStream_t s, const uint32_t *sys_off, int n_sys) {
    const uint32_t rows = (n + RANK_ROWS - 1) / RANK_ROWS;
    if (sys_off && n_sys > 1) k_sort_small<true><<<rows, RANK_THREADS, 0, s>>>(key, val, key_out, val_out, n, sys_off, n_sys);
    else k_sort_small<false><<<rows, RANK_THREADS, 0, s>>>(key, val, key_out, val_out, n, sys_off, 1);
}

void radix_sort(uint64_t *key_a, uint32_t *val_a, uint64_t *key_b, uint32_t *val_b,
                uint32_t n, int lo_bit, int hi_bit, uint32_t *hist, uint32_t *tmp, hipStream_t s,
                const uint32_t *sys_off, int n_sys) {
    if (n == 0) return;
    if (!sys_off) n_sys = 1;
    // ranks up to SMALL_MAX, the sample sort up to SAMPLE_MAX, radix passes above
    if (n <= SMALL_MAX) {
        sort_small(key_a, val_a, key_b, val_b, n, s, sys_off, n_sys);
        k_copy_pairs<<<(n + 255) / 256, 256, 0, s>>>(key_b, val_b, key_a, val_a, n);
        return;
    }
    if (n <= SAMPLE_MAX) {
        const bool sys = n_sys > 1;
        const SamplePlan plan = sample_plan(n, sys);
        const SampleLayout L = ss_layout(n, plan, hist);
        const uint32_t rows = (L.buckets * L.per + RANK_ROWS - 1) / RANK_ROWS;
        k_ss_gather<<<(L.buckets * L.per + 255) / 256, 256, 0, s>>>(key_a, val_a, sys_off, n_sys, L, key_b, val_b);
        if (sys) k_ss_rank<true><<<rows, RANK_THREADS, 0, s>>>(key_b, val_b, L);
        else k_ss_rank<false><<<rows, RANK_THREADS, 0, s>>>(key_b, val_b, L);
        k_ss_hist<<<L.tiles, SS_THREADS, 0, s>>>(key_a, val_a, n, sys_off, n_sys, L);
        scan_u32(L.hist, L.hist, L.buckets * L.tiles, tmp, s);
        k_ss_scatter<<<L.tiles, SS_THREADS, 0, s>>>(key_a, val_a, key_b, val_b, n, L);
        auto last = [&](auto kernel) {
            kernel<<<L.buckets, SS_SORT, 0, s>>>(key_b, val_b, key_a, val_a, n, sys_off, n_sys, L);
        };
        if (plan.capacity > CAP_NARROW) sys ? last(k_ss_sort<CAP_WIDE_SYS, true>) : last(k_ss_sort<CAP_WIDE, false>);
        else sys ? last(k_ss_sort<CAP_NARROW, true>) : last(k_ss_sort<CAP_NARROW, false>);
        return;
    }
    uint32_t nb = (n + RS_TILE - 1) / RS_TILE;
    uint64_t *ki = key_a, *ko = key_b;
    uint32_t *vi = val_a, *vo = val_b;
    int passes = 0;
    auto pass = [&](bool sys, int sh) {
        if (sys) {
            k_radix_hist<true><<<nb, RS_THREADS, 0, s>>>(ki, vi, n, sh, hist, nb, sys_off, n_sys);
        } else {
            k_radix_hist<false><<<nb, RS_THREADS, 0, s>>>(ki, vi, n, sh, hist, nb, sys_off, n_sys);
        }
        scan_u32(hist, hist, nb * 256, tmp, s);
        if (sys) {
            k_radix_scatter<true><<<nb, RS_THREADS, 0, s>>>(ki, vi, ko, vo, n, sh, hist, nb, sys_off, n_sys);
        } else {
            k_radix_scatter<false><<<nb, RS_THREADS, 0, s>>>(ki, vi, ko, vo, n, sh, hist, nb, sys_off, n_sys);
        }
        uint64_t *kt = ki; ki = ko; ko = kt;
        uint32_t *vt = vi; vi = vo; vo = vt;
        ++passes;
    };
    for (int sh = lo_bit; sh < hi_bit; sh += 8) pass(false, sh);
    // systems are the most significant digit: a final stable pass per 8 bits of system index
    if (sys_off && n_sys > 1)
        for (int sh = 0; (n_sys - 1) >> sh; sh += 8) pass(true, sh);
    if (passes & 1) k_copy_pairs<<<(n + 255) / 256, 256, 0, s>>>(ki, vi, key_a, val_a, n);
}

}  // namespace bhk
