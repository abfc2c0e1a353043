// Work plan of a batch: configurations grouped into classes (by size or by number of pairs, so that each
// class gets the kernel variant and group size that fit it) and, inside a class, ordered from most to least work, so the
// longest-running configurations start first.  Built on the device, in one block for small batches and by four
// small kernels for larger ones; no host sync.
#pragma once

#include "prs_device.h"

namespace prs {

constexpr int kClasses = 6;          // bi-greedy: five group sizes and the general kernel; uni-greedy: six group sizes (schedules of large machines use 0, 1, 2 and the last)
constexpr int kWorkBuckets = 40;     // floor(log2(work)) buckets, heaviest first
constexpr int kRetryClass = kClasses; // pseudo class: configurations handed back to the general kernel
constexpr int kWideClass = kClasses;  // uni-greedy completion times: machines large enough for a block of their own
constexpr int kLargeClass = kClasses + 1;   // uni-greedy: the classes 0 .. kClasses - 1 again, for machines of more than large_p processors
constexpr int kPlanClasses = kLargeClass + kClasses;

struct PlanHeader {
    unsigned long long ticket[kPlanClasses];
    // The heaviest configurations of the last class (at least 2^giant_log2 pairs) come first in its order; the
    // uni-greedy kernels run them on whole wavefronts and draw them from a ticket counter of their own ([1]: large machines).
    unsigned long long ticket_giant[2];
    int32_t giant_count[2];
    int32_t large_left;                           // large machines that are not done
    int32_t several;                              // bi-greedy: 1 if some configuration requests more than one segment
    int32_t class_begin[kPlanClasses];
    int32_t class_count[kPlanClasses];
    int32_t place[kPlanClasses * kWorkBuckets];   // configurations per bucket, then where the next one of the bucket goes
};
constexpr int kGiantLog2 = 23;
enum ClassPart { kWholeClass = 0, kGiantPart = 1, kRestPart = 2 };

// By size (by_work == 0): class k holds p <= limits.p[0][k]; the last class the rest and every configuration
// with more than q segments.
// By work (by_work != 0): class k holds the configurations with at most work[k] pairs and p[k] processors, the last class
// the rest.  Machines of more than large_p processors (0: none) have classes of their own, with the limits [1] instead of [0].
struct ClassLimits {
    int32_t p[2][kClasses - 1];
    int32_t q;
    int32_t by_work;
    int32_t large_p;
    int64_t work[2][kClasses - 1];
    int32_t giant_log2[2];       // configurations of the last class with at least 2^giant_log2 pairs are "giant"
    int32_t lanes_log2[2];       // by_work only: 1: class k has 2^k lanes per configuration, and none gets more than it has segments
    int32_t lane_p;              // by_work only: the first set's class k holds at most 2^k times as many processors (0: no such limit)
    int32_t wide_p;              // by_work only: machines of at least this many processors form the class kWideClass (0: none)
};

struct PlanLaunch {
    ConfigArrays cfg;
    int64_t n;
    int32_t p_max, q_max;
    int cost;
    ClassLimits limits;
    PlanHeader *header;
    int32_t *order;
    hipStream_t stream;
};

hipError_t launch_plan(const PlanLaunch &L);

__host__ __device__ inline size_t plan_header_bytes() { return (sizeof(PlanHeader) + 255) / 256 * 256; }

}  // namespace prs
