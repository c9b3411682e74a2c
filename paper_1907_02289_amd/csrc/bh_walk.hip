// bh_walk.hip -- interaction lists, Iwasawa et al. (2019) Sec. 4.2 step (3d):
// the tree is traversed once per group of neighbouring particles (the group
// variant of the walk), producing the list of tree nodes and the list of
// particles (as leaves) that act on the group; the lists are kept and reused
// over several steps (the persistent interaction list of Sec. 4.2).
//
// One wavefront walks one group.  The traversal is breadth first: the 64
// lanes test 64 frontier nodes at a time and ballots / a wave prefix sum
// compact the three outcomes (accepted node -> node list, rejected leaf ->
// particle list, rejected internal node -> its children join the next
// frontier).  Frontier order is ascending node id at every level, so both
// lists come out in ascending node id without a sort.
//
// Opening test (the paper states none; reading): a node is accepted when it
// lies outside the group's grid box and side < theta * distance from the
// node's centre to the box, evaluated in doubled integer grid units with a
// single FP64 multiply, so every device decides exactly alike.  On
// cylindrical tree coordinates (Sec. 4.3) the phi axis is periodic with one
// turn = 2^21 grid units: its distance is that of the node's nearest image
// (a node and a group box inside one turn overlap only directly).
#include <algorithm>

#include "bh_learned.hpp"

namespace {

constexpr int WALK_TPB = 256;
constexpr int WALK_LFRONT = 512;    // frontier entries kept in LDS per wave and buffer

// The opening test, in 32-bit integers with the squared distance summed in
// FP64: every doubled coordinate and gap is below 2^24 and every square below
// 2^47, so each step is exact and the decision is that of 64-bit integers, bit
// for bit, in about half the instructions.
__device__ __forceinline__ int gap2(int C, int gl2, int gh2) { return max(0, max(gl2 - C, C - gh2)); }

__device__ __forceinline__ bool accept_cell(int4 glo, int4 ghi, int Lx, int Ly, int Lz, int level, double th2,
                                            bool periodic) {
    const int s = 1 << (BH_MAXLEVEL - level);
    const int L[3] = {Lx, Ly, Lz};
    const int gl[3] = {glo.x, glo.y, glo.z}, gh[3] = {ghi.x, ghi.y, ghi.z};
    constexpr int TURN2 = 2 << BH_MAXLEVEL;                 // one turn of phi, doubled units
    bool disjoint = false;
    double d2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        disjoint |= (L[a] + s <= gl[a]) || (L[a] >= gh[a]);
        const int C = 2 * L[a] + s;
        int da = gap2(C, 2 * gl[a], 2 * gh[a]);
        if (a == 0 && periodic)
            da = min(da, min(gap2(C - TURN2, 2 * gl[a], 2 * gh[a]), gap2(C + TURN2, 2 * gl[a], 2 * gh[a])));
        d2 = fma((double)da, (double)da, d2);
    }
    const double s2 = (double)(4 * s) * (double)s;          // (2 s)^2
    return disjoint && (s2 < th2 * d2);
}

// Number of set bits of m in the lanes below this one.
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Exclusive prefix sum over the lanes of a value in 0..15, and the wave
// total, from four ballots (no cross-lane data movement).
__device__ __forceinline__ uint32_t wave_excl_small(uint32_t v, uint32_t &tot) {
    uint32_t pre = 0;
    tot = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t b = __ballot((v >> k) & 1u);
        pre += mbcnt(b) << k;
        tot += (uint32_t)__popcll(b) << k;
    }
    return pre;
}

// Per-group constants of the learned rule.
struct GroupCtx {
    int4 glo, ghi;
    double4 cen;
    double rad, amin, Msys;
};

// Node v for a group under the learned and the enumerating rule.  LEARNED:
// below theta_min accept, at or above theta_max open, in between the network
// (single-particle nodes accepted, nodes above the count cap: the theta test).
// ENUMERATE: the theta_min test; *cand reports whether (group, v) lies in the
// band and is a training candidate.  For NETWORK f and below are the network's
// inputs and the value its output has to stay below.
enum Verdict { OPEN, ACCEPT, NETWORK };

__device__ __forceinline__ Verdict judge(const DevState &d, const GroupCtx &gc, uint32_t v, int4 wr, bool *cand,
                                         float f[MLP_NIN], double *below) {
    const int level = (int)((uint32_t)wr.x >> 24);
    const int Lx = wr.x & 0xffffff, Ly = wr.y & 0xffffff, Lz = wr.z;
    if (accept_cell(gc.glo, gc.ghi, Lx, Ly, Lz, level, d.th2_min, false)) return ACCEPT;
    if (!accept_cell(gc.glo, gc.ghi, Lx, Ly, Lz, level, d.th2_max, false)) return OPEN;
    const uint32_t cnt = d.nd_count[v];
    if (d.walk_mode == WALK_ENUMERATE) {
        *cand = cnt >= 2 && cnt <= d.count_cap;
        return OPEN;
    }
    if (cnt == 1) return ACCEPT;
    if (cnt > d.count_cap) return accept_cell(gc.glo, gc.ghi, Lx, Ly, Lz, level, d.th2, false) ? ACCEPT : OPEN;
    const double4 mom = d.nd_mom[v];
    const PairGeom pg =
        pair_features(mom, box_ratio2(gc.glo, gc.ghi, Lx, Ly, Lz, level), d.nd_qn[v], gc.cen, gc.rad, gc.Msys);
    for (int k = 0; k < MLP_NIN; ++k) f[k] = pg.f[k];
    *below = accept_below(pg, mom.w, gc.amin, d.tau, d.G);
    return NETWORK;
}

// Rounds: four consecutive groups, one per wave of a block.  Runs of WALK_CHUNK
// rounds go to the XCDs in turn: walk_share is the most that one XCD has.
constexpr uint32_t WALK_CHUNK = 8;
__host__ __device__ inline uint32_t walk_rounds(uint32_t n_groups) { return (n_groups + WALK_TPB / 64 - 1) / (WALK_TPB / 64); }
__host__ __device__ inline uint32_t walk_share(uint32_t rounds) {
    return (rounds + 8 * WALK_CHUNK - 1) / (8 * WALK_CHUNK) * WALK_CHUNK;
}

// Persistent blocks of four waves, one group per wave and round.  What
// bounded an earlier form was neither the walk's memory traffic nor its
// arithmetic but atomics on one cache line: each wave popped its groups from
// a counter and reserved its list space with four more returning atomics per
// group, and same-line atomics of the whole chip are served one per 12 ns
// (measured: walk time / number of atomics = 11.6..12.4 ns from 172 to
// 138,763 groups).  Now a block takes rounds of four consecutive groups, the
// first by its number, further ones from its XCD's counter; its waves reserve
// list space together, the two pools and the next round with one instruction on
// three cache lines, and the interaction total is summed in registers and added
// once per block.
// Blocks are dealt to the eight XCDs in turn, and so are runs of WALK_CHUNK
// rounds along the curve: neighbouring groups open the same nodes, which stay in
// that XCD's L2, while a region of long walks (a dense centre, one large system
// among small ones) spreads over all XCDs.  One contiguous eighth per XCD with
// its rounds dealt by block number left XCDs idle: Plummer sphere of 2^22
// particles, theta 0.1, 121 -> 100 ms; of 2^21 with 3000 rings of 100 beside it
// 55.9 -> 39.9 ms; ring of 2^22 in 400,633 groups, theta 0.3, 3.5 -> 2.8 ms.
// Runs of 4 rounds take the same time, runs of 32 up to 5% more.
// The next 64 nodes are loaded before the current 64 are tested; a leaf's
// particle count rides in the node record, so a visit is one 16-byte load.
// Kernel time with the counter per group and now: 172 groups (4096-particle ring)
// 105 -> 14 us, 9,311 groups (200k, theta 0.2) 560 -> 78 us, 15,739 groups (2^20,
// theta 0.5) 863 -> 89 us, 64 Plummer spheres 878 -> 200 us; with 60,447 groups of
// 10^4-entry lists (2^24, theta 0.0865) the visits themselves take the time,
// 6.0 -> 5.7 ms (stage, one card in turn).
// GEO: the instance of the geometric rule, without the registers of the
// network.  The other one has 227 (two waves per SIMD, as many as are launched):
// held to 168 or 128 its walks took 3% and 10% longer.
template <bool GEO>
__global__ void __launch_bounds__(WALK_TPB, (GEO ? 8 : 2)) k_walk(DevState d) {
    constexpr uint32_t WPB = WALK_TPB / 64;
    const uint32_t wib = threadIdx.x >> 6;
    const uint32_t wave = blockIdx.x * WPB + wib;
    const int lane = __lane_id();
    const uint64_t lt = lanemask_lt();
    const uint32_t F = d.walk_front_cap, P = d.walk_list_cap;
    uint32_t *fa = d.walk_scratch + (size_t)wave * (2 * (size_t)F + 2 * (size_t)P);
    uint32_t *fb = fa + F;
    uint32_t *pcb = fb + F;
    uint32_t *ppb = pcb + P;
    const uint32_t ng = d.cnt->n_groups;
    const uint32_t n_nodes = d.cnt->lvl_off[BH_NLEVELS];
    // the first WALK_LFRONT entries of each frontier live in LDS, the rest at
    // the same index in the wave's global scratch
    __shared__ uint32_t lfront[WPB][2][WALK_LFRONT];
    uint32_t *la = lfront[wib][0], *lb = lfront[wib][1];
    const bool learned = !GEO && d.walk_mode == WALK_LEARNED;
    WaveNet net;
    __shared__ alignas(16) float s_net[GEO ? 1 : WNET_LDS];
    if constexpr (!GEO) {
        if (learned) {
            net = wave_net_load(d.mlp);
            for (int k = threadIdx.x; k < WNET_LDS; k += WALK_TPB) s_net[k] = wave_net_lds_entry(d.mlp, k);
        }
        __syncthreads();
    }
    __shared__ uint32_t s_len[WPB][2];             // list lengths of the block's four groups
    __shared__ unsigned long long s_at[3];         // the block's starts in the two pools, and its next round
    __shared__ unsigned long long s_cost[WPB];
    unsigned long long cost_sum = 0;

    const uint32_t rounds = walk_rounds(ng), xcd = blockIdx.x & 7u, bx = gridDim.x >> 3;    // gridDim.x is a multiple of 8
    const bool more = bx < walk_share(rounds);     // rounds beyond one per block
    for (uint32_t k = blockIdx.x >> 3;;) {
        const uint32_t round = (k / WALK_CHUNK * 8 + xcd) * WALK_CHUNK + k % WALK_CHUNK;
        if (round >= rounds) break;
        const uint32_t g0 = round * WPB;
        const uint32_t g = g0 + wib;
        const bool has = g < ng;
        uint32_t npc = 0, npp = 0, n_part = 0;
        unsigned long long pp_particles = 0;
        bool skip = !has;       // no lists to store (no group, or its walk was cut short)
        // the enumerating walk visits only the sampled groups and stores no lists
        const bool enumerate = !GEO && d.walk_mode == WALK_ENUMERATE;
        const bool record = enumerate && (g % d.group_stride) == 0;
        if (has && !(enumerate && !record)) {
            const GroupInfo gi = d.grp[g];
            n_part = gi.count;
            GroupCtx gc;
            gc.glo = d.g_lo[g];
            gc.ghi = d.g_hi[g];
            if constexpr (!GEO) {
                gc.cen = d.g_cen[g];
                gc.rad = d.g_rad[g];
                gc.amin = learned ? d.g_amin[g] : 0.0;
                gc.Msys = d.nd_mom[gi.sys].w;
            }
            uint32_t *cur = fa, *nxt = fb;
            uint32_t *lcur = la, *lnxt = lb;
            if (lane == 0) lcur[0] = gi.sys;         // root of the group's system
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint32_t ncur = 1;
            unsigned long long pp_lane = 0;          // this lane's share, summed once per group
            bool ovf = false, bound = false;
            // A walk of a well-formed tree descends one level per frontier and
            // visits every node at most once; a frontier beyond the deepest level
            // or more visits than nodes can only come from a malformed tree, and
            // ends the walk with a flag instead of running on.
            uint32_t levels = 0;
            unsigned long long visits = 0;
            while (ncur > 0 && !ovf && !bound) {
                visits += ncur;
                if (++levels > (uint32_t)BH_NLEVELS || visits > (unsigned long long)n_nodes) {
                    bound = true;
                    break;
                }
                uint32_t nnext = 0;
                auto front = [&](uint32_t k) -> uint32_t {
                    return k < (uint32_t)WALK_LFRONT ? lcur[k] : cur[k];
                };
                uint32_t v_next = (uint32_t)lane < ncur ? front(lane) : 0u;
                int4 wr_next = (uint32_t)lane < ncur ? d.nd_walk[v_next] : make_int4(0, 0, 0, 0);
                for (uint32_t base = 0; base < ncur; base += 64) {
                    const uint32_t k = base + lane;
                    const bool valid = k < ncur;
                    const uint32_t v = v_next;
                    const int4 wr = wr_next;
                    const uint32_t kn = k + 64;
                    if (kn < ncur) {
                        v_next = front(kn);
                        wr_next = d.nd_walk[v_next];
                    }
                    const int nch = (int)((uint32_t)wr.y >> 24);
                    bool is_cand = false;
                    bool acc;
                    if constexpr (GEO) {
                        acc = valid && accept_cell(gc.glo, gc.ghi, wr.x & 0xffffff, wr.y & 0xffffff, wr.z,
                                                   (int)((uint32_t)wr.x >> 24), d.th2, d.cyl_r > 0.0);
                    } else {
                        float f[MLP_NIN] = {0.0f, 0.0f, 0.0f, 0.0f};
                        double below = 0.0;
                        const Verdict vd = valid ? judge(d, gc, v, wr, &is_cand, f, &below) : OPEN;
                        acc = vd == ACCEPT;
                        if (__ballot(vd == NETWORK)) {
                            const float y = wave_net_forward(net, s_net, f);
                            if (vd == NETWORK) acc = (double)y < below;
                        }
                    }
                    if constexpr (!GEO) {
                        is_cand = is_cand && valid && record;
                        const uint64_t mc = __ballot(is_cand);
                        if (mc) {
                            unsigned long long at = 0;
                            if (lane == 0) at = atomicAdd(&d.cnt->cand_used, (unsigned long long)__popcll(mc));
                            at = __shfl(at, 0, 64) + (unsigned long long)__popcll(mc & lt);
                            if (is_cand && at < d.cand_cap) d.cand[at] = make_uint2(g, v);
                        }
                    }
                    const bool is_pp = valid && !acc && nch == 0;
                    const uint32_t nopen = (valid && !acc && nch > 0) ? (uint32_t)nch : 0u;

                    const uint64_t mpc = __ballot(acc);
                    const uint64_t mpp = __ballot(is_pp);
                    const uint32_t opc = npc + mbcnt(mpc);
                    const uint32_t opp = npp + mbcnt(mpp);
                    if (acc && opc < P && !enumerate) pcb[opc] = v;
                    if (is_pp && opp < P && !enumerate) ppb[opp] = v;
                    if (is_pp) pp_lane += (uint32_t)wr.w;       // a leaf's record holds its particle count
                    npc += (uint32_t)__popcll(mpc);
                    npp += (uint32_t)__popcll(mpp);
                    uint32_t tot;
                    const uint32_t o = nnext + wave_excl_small(nopen, tot);
                    for (uint32_t c = 0; c < nopen; ++c) {
                        const uint32_t q = o + c;
                        if (q < (uint32_t)WALK_LFRONT) lnxt[q] = (uint32_t)wr.w + c;
                        else if (q < F) nxt[q] = (uint32_t)wr.w + c;
                    }
                    nnext += tot;
                }
                if (nnext > F || (!enumerate && (npc > P || npp > P))) ovf = true;
                // the next frontier is read by other lanes of this wave than wrote it: LDS
                // accesses of a wave complete in order; entries in global memory need the wait
                if (nnext > (uint32_t)WALK_LFRONT) __threadfence_block();
                else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                uint32_t *t = cur; cur = nxt; nxt = t;
                t = lcur; lcur = lnxt; lnxt = t;
                ncur = nnext;
            }
            if (bound) {
                if (lane == 0) atomicOr(&d.cnt->flags[FLAG_WALK_BOUND], 1u);
            } else if (ovf) {
                if (lane == 0) {
                    atomicOr(&d.cnt->flags[FLAG_WALK_OVF], 1u);
                    atomicMax(&d.cnt->walk_need_front, ncur);
                    if (!enumerate) atomicMax(&d.cnt->walk_need_list, max(npc, npp));
                }
            } else {
                pp_particles = wave_sum(pp_lane);
            }
            skip = bound || ovf || enumerate;
        } else {
            skip = true;
        }
        if (skip) npc = npp = 0;
        if (lane == 0) {
            s_len[wib][0] = npc;
            s_len[wib][1] = npp;
        }
        __syncthreads();
        if (threadIdx.x < 3) {                  // three cache lines in one instruction
            unsigned long long sum = more ? 1 : 0;
            if (threadIdx.x < 2) {
                sum = 0;
                for (uint32_t q = 0; q < WPB; ++q) sum += s_len[q][threadIdx.x];
            }
            unsigned long long *head = threadIdx.x == 0   ? &d.cnt->pc_used
                                       : threadIdx.x == 1 ? &d.cnt->pp_used
                                                          : &d.cnt->walk_round[xcd].taken;
            s_at[threadIdx.x] = sum ? atomicAdd(head, sum) : 0ull;
        }
        __syncthreads();
        unsigned long long at_pc = s_at[0], at_pp = s_at[1];
        k = __builtin_amdgcn_readfirstlane((uint32_t)s_at[2]) + bx;     // past the end when there is no more
        for (uint32_t q = 0; q < wib; ++q) {
            at_pc += s_len[q][0];
            at_pp += s_len[q][1];
        }
        const bool fit = !skip && (at_pc + npc <= d.pc_cap) && (at_pp + npp <= d.pp_cap);
        if (fit) {
            __threadfence_block();              // the scratch lists, written by other lanes
            for (uint32_t q = lane; q < npc; q += 64) d.pc_pool[at_pc + q] = pcb[q];
            for (uint32_t q = lane; q < npp; q += 64) d.pp_pool[at_pp + q] = ppb[q];
        } else if (lane == 0 && !skip) {
            atomicOr(&d.cnt->flags[FLAG_POOL_OVF], 1u);
        }
        const unsigned long long cost = skip ? 0ull : (unsigned long long)n_part * (pp_particles + npc);
        cost_sum += cost;
        if (lane == 0 && has) {
            d.g_pc_off[g] = fit ? at_pc : 0ull;
            d.g_pc_len[g] = fit ? npc : 0u;
            d.g_pp_off[g] = fit ? at_pp : 0ull;
            d.g_pp_len[g] = fit ? npp : 0u;
            d.g_cost[g] = cost;
        }
        __syncthreads();                        // s_len and s_at are free for the next round
    }
    if (lane == 0) s_cost[wib] = cost_sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (uint32_t k = 0; k < WPB; ++k) sum += s_cost[k];
        if (sum) atomicAdd(&d.cnt->interactions, sum);
    }
}

__global__ void k_walk_reset(DevState d) {
    if (threadIdx.x == 0 && blockIdx.x == 0) reset_walk_counters(d);
}

// Work order for the force kernel: groups by descending interaction count
// (the list-length ordering of the paper's load balance, Sec. 4.6), in
// classes of half an octave of cost; inside a class, ascending group id,
// i.e. along the Morton curve, so that the groups in flight at one time are
// neighbours whose lists share most of their sources in L2.  A counting sort of
// the groups' work items: items of each class per tile of groups, then every tile's block sums the table up to
// itself and writes the force kernel's records in place.  At most ORDER_TILES
// tiles keep the table at 32 KB.  (A radix pass over (class, id) keys and the
// records were 7 launches, 4 below 8192 groups.)  What bounds these sizes is
// launches and the host between them: with the four launches of the groups, the
// sort's copy and one of three counter reads less, a call at 4096 particles
// went from 286 to 232 us, a 2^20 step from 1.43 to 1.33 ms.
constexpr uint32_t ORDER_TILES = 64;
constexpr uint32_t ORDER_CLASSES = 128;
constexpr uint32_t ORDER_TPB = 256;
static_assert(ORDER_TILES * ORDER_CLASSES <= bhk::ORDER_WORDS, "the table lies in d.hist");

__device__ __forceinline__ uint32_t order_class(const DevState &d, uint32_t g) {
    const unsigned long long c = d.g_cost[g];
    const uint32_t cls = c ? (uint32_t)(2.0 * log2((double)c)) : 0u;
    return 127u - (cls < 127u ? cls : 127u);              // largest cost first
}

__device__ __forceinline__ uint32_t item_count(const GroupInfo &gi) {
    return (gi.count + ITEM_PARTICLES - 1) / ITEM_PARTICLES;
}

__global__ void __launch_bounds__(ORDER_TPB) k_order_count(DevState d, uint32_t ng, uint32_t tile) {
    __shared__ uint32_t cnt[ORDER_CLASSES];
    if (threadIdx.x < ORDER_CLASSES) cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t b = blockIdx.x * tile, e = min(b + tile, ng);
    for (uint32_t g = b + threadIdx.x; g < e; g += ORDER_TPB) atomicAdd(&cnt[order_class(d, g)], item_count(d.grp[g]));
    __syncthreads();
    if (threadIdx.x < ORDER_CLASSES) d.hist[threadIdx.x * gridDim.x + blockIdx.x] = cnt[threadIdx.x];
}

__global__ void __launch_bounds__(ORDER_TPB) k_order_place(DevState d, uint32_t ng, uint32_t tile) {
    __shared__ uint32_t start[ORDER_CLASSES], total[ORDER_CLASSES], cnt[ORDER_TPB / 64][ORDER_CLASSES];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    // this tile's start in each class: the smaller classes' items and those of the tiles before
    if (threadIdx.x < ORDER_CLASSES) {
        uint32_t before = 0, all = 0;
#pragma unroll 8
        for (uint32_t t = 0; t < gridDim.x; ++t) {
            const uint32_t c = d.hist[threadIdx.x * gridDim.x + t];
            before += t < blockIdx.x ? c : 0u;
            all += c;
        }
        start[threadIdx.x] = before;
        const uint32_t inc = wave_incl_scan(all);
        total[threadIdx.x] = inc - all;
        if (lane == 63) cnt[w][0] = inc;
    }
    __syncthreads();
    if (threadIdx.x < ORDER_CLASSES) start[threadIdx.x] += total[threadIdx.x] + (w ? cnt[0][0] : 0u);
    if (blockIdx.x == 0 && threadIdx.x == 0) d.cnt->n_items = cnt[0][0] + cnt[1][0];
    const uint32_t b = blockIdx.x * tile, e = min(b + tile, ng);
    for (uint32_t g0 = b; g0 < e; g0 += ORDER_TPB) {
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < ORDER_TPB / 64 * ORDER_CLASSES; k += ORDER_TPB) (&cnt[0][0])[k] = 0;
        __syncthreads();
        const uint32_t g = g0 + threadIdx.x;
        const bool on = g < e;
        const GroupInfo gi = on ? d.grp[g] : GroupInfo{0, 0, 0, 0};
        const uint32_t o = on ? order_class(d, g) : 0u, items = on ? item_count(gi) : 0u;
        // items of the same class in the lanes below: class after class
        uint32_t rank = 0;
        for (uint64_t left = __ballot(on); left;) {
            const uint32_t cls = __shfl(o, __ffsll((unsigned long long)left) - 1, 64);
            const bool mine = on && o == cls;
            const uint32_t inc = wave_incl_scan(mine ? items : 0u);
            if (mine) rank = inc - items;
            if (lane == 63) cnt[w][cls] = inc;
            left &= ~__ballot(mine);
        }
        __syncthreads();
        if (on) {
            uint32_t at = start[o] + rank;
            for (int k = 0; k < w; ++k) at += cnt[k][o];
            const double4 c = d.g_cen[g];
            const double m0 = d.sys_m0[gi.sys];
            ForceItem it{c.x, c.y, c.z, m0, m0 > 0.0 ? 1.0 / m0 : 1.0, d.g_pc_off[g], d.g_pp_off[g], d.g_pc_len[g],
                         d.g_pp_len[g], gi.begin, 0};
            for (uint32_t k = 0; k < items; ++k, it.begin += ITEM_PARTICLES) {
                it.count = min(ITEM_PARTICLES, gi.count - k * ITEM_PARTICLES);
                d.force_items[at + k] = it;
            }
        }
        __syncthreads();
        if (threadIdx.x < ORDER_CLASSES)
            for (int k = 0; k < (int)(ORDER_TPB / 64); ++k) start[threadIdx.x] += cnt[k][threadIdx.x];
    }
}

}  // namespace

namespace bhk {

void walk(const DevState &d, uint32_t n_groups, bool reset, hipStream_t s) {
    if (reset) k_walk_reset<<<1, 64, 0, s>>>(d);
    if (n_groups == 0) return;
    // as many blocks as stay resident (and have scratch), one per round when there are
    // fewer rounds; a multiple of 8, one share per XCD
    const uint32_t waves = d.walk_mode == WALK_GEOMETRIC ? d.walk_waves : d.walk_waves_net;
    const uint32_t blocks = std::min(waves / (WALK_TPB / 64) & ~7u, 8 * walk_share(walk_rounds(n_groups)));
    if (d.walk_mode == WALK_GEOMETRIC)
        k_walk<true><<<blocks, WALK_TPB, 0, s>>>(d);
    else
        k_walk<false><<<blocks, WALK_TPB, 0, s>>>(d);
}

void order_groups(const DevState &d, uint32_t n_groups, hipStream_t s) {
    if (n_groups == 0) return;
    const uint32_t per = (n_groups + ORDER_TILES - 1) / ORDER_TILES;
    const uint32_t tile = (per + ORDER_TPB - 1) / ORDER_TPB * ORDER_TPB, tiles = (n_groups + tile - 1) / tile;
    k_order_count<<<tiles, ORDER_TPB, 0, s>>>(d, n_groups, tile);
    k_order_place<<<tiles, ORDER_TPB, 0, s>>>(d, n_groups, tile);
}

}  // namespace bhk
