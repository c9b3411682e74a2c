// bh_sort_plan.hpp -- which way a sort of n pairs takes and the sizes of the
// sample sort: host arithmetic only.
#pragma once
#include <stdint.h>

namespace bhk {

constexpr uint32_t SMALL_MAX = 8192;            // places counted by comparison up to here
constexpr uint32_t SAMPLE_MAX = 5u << 19;       // sample sort up to here (2.6e6 pairs), radix passes above
constexpr uint32_t BUCKETS_MAX = 1024;

// The sample sort: buckets, sampled pairs per bucket, and the pairs that a
// bucket's block holds in LDS; larger buckets are sorted by their block over
// memory, while the chip waits for it.  In randomly ordered input a bucket is
// the sum of `per` gaps between sampled pairs, so its share of the n pairs is
// Beta(per, buckets per + 1 - per) distributed and the expected number of
// buckets above the capacity follows.  Up to 2^20 pairs the capacity is 4096,
// four times the average: 1e-4 of the sorts at 8 per bucket.  Above, the LDS of
// two blocks per CU has room for 7680 pairs, 6144 with their systems, down to
// 2.4 times the average: at 8 per bucket 0.05 and 1.3 buckets of a sort at
// SAMPLE_MAX were larger.  More sampled pairs narrow the distribution, and their
// ranking grows with the square (2.2e6 pairs of 64 systems: 54 us at 16 per
// bucket), so as many are taken as the capacity asks for: 8 down to 3.5 times
// the average (5e-3), 12 down to 2.8 times (5e-3), 16 below (0.015).
struct SamplePlan {
    uint32_t buckets, per, capacity;
};

constexpr uint32_t CAP_NARROW = 4096, CAP_WIDE = 7680, CAP_WIDE_SYS = 6144;

inline SamplePlan sample_plan(uint32_t n, bool several_systems) {
    const uint32_t want = (n + 1023) / 1024;
    const uint32_t buckets = want < 8 ? 8u : (want > BUCKETS_MAX ? BUCKETS_MAX : want);
    const uint32_t capacity = n <= (1u << 20) ? CAP_NARROW : several_systems ? CAP_WIDE_SYS : CAP_WIDE;
    const uint64_t room = 10ull * capacity * buckets;       // ten times capacity / average, times n
    return {buckets, room >= 35ull * n ? 8u : room >= 28ull * n ? 12u : 16u, capacity};
}

}  // namespace bhk
