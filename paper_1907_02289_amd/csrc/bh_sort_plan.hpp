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
// buckets above the capacity follows: 8 per bucket hold 4096 at n = 2^20 (four
// times the average) but for 1e-4 of the sorts.  Above, the LDS of two blocks
// per CU has room for 7680 pairs, 6144 with their systems, down to 2.4 times
// the average: with 8 per bucket 0.05 and 1.3 buckets of a sort at SAMPLE_MAX
// were larger, with 16 it is 3e-5 and 0.015.
struct SamplePlan {
    uint32_t buckets, per, capacity;
};

constexpr uint32_t CAP_NARROW = 4096, CAP_WIDE = 7680, CAP_WIDE_SYS = 6144;

inline SamplePlan sample_plan(uint32_t n, bool several_systems) {
    const uint32_t b = (n + 1023) / 1024;
    const bool wide = n > (1u << 20);
    return {b < 8 ? 8u : (b > BUCKETS_MAX ? BUCKETS_MAX : b), wide ? 16u : 8u,
            !wide ? CAP_NARROW : several_systems ? CAP_WIDE_SYS : CAP_WIDE};
}

}  // namespace bhk
