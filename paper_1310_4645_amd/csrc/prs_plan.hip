#include "prs_plan.h"

namespace prs {

template <typename T>
__device__ __forceinline__ int plan_bucket(const ConfigArrays &cfg, int64_t i, int32_t p_max, int32_t q_max,
                                           const ClassLimits &lim)
{
    const Config<T> c = decode_config<T>(cfg, i, p_max, q_max);
    if (c.status != PRS_CFG_OK) return kWorkBuckets - 1;                 // nothing to do: lightest bucket of class 0
    const int64_t work = static_cast<int64_t>(c.p - 1) * c.q;
    int cls = kClasses - 1;
    if (lim.by_work) {
        const bool large = lim.large_p > 0 && c.p > lim.large_p;
        for (int k = kClasses - 2; k >= 0; --k)
            if (work <= lim.work[large ? 1 : 0][k] && c.p <= lim.p[large ? 1 : 0][k]) cls = k;
        if (lim.lanes_log2[large ? 1 : 0]) { const int enough = ceil_log2(c.q); cls = cls < enough ? cls : enough; }
        if (lim.lane_p > 0 && !large) { const int least = ceil_log2((c.p + lim.lane_p - 1) / lim.lane_p); cls = cls > least ? cls : least; }
        if (large) cls += kLargeClass;
        if (lim.wide_p > 0 && c.p >= lim.wide_p && cfg.comp_m == 0) cls = kWideClass;
    } else {
        for (int k = kClasses - 2; k >= 0; --k)
            if (c.p <= lim.p[0][k] && c.q <= lim.q) cls = k;
    }
    int lg = 63 - __builtin_clzll(static_cast<unsigned long long>(work) | 1ULL);
    if (lg > kWorkBuckets - 1) lg = kWorkBuckets - 1;
    return cls * kWorkBuckets + (kWorkBuckets - 1 - lg);
}

__global__ void plan_clear(PlanHeader *h)
{
    const int i = threadIdx.x;
    if (i < kPlanClasses) { h->ticket[i] = 0ULL; h->class_begin[i] = 0; h->class_count[i] = 0; }
    if (i < 2) { h->giant_count[i] = 0; h->ticket_giant[i] = 0ULL; }
    if (i == 0) { h->large_left = 0; h->several = 0; }
    for (int k = i; k < kPlanClasses * kWorkBuckets; k += blockDim.x) h->place[k] = 0;
}

constexpr int kPlanThreads = 256;
constexpr int kPlanBins = kPlanClasses * kWorkBuckets;

// Both passes count inside the block first (LDS) and touch the global counters once per block and bin: with one
// global atomic per configuration, a batch of millions spends its time queueing on a few dozen addresses.
template <typename T>
__global__ __launch_bounds__(kPlanThreads) void plan_hist(ConfigArrays cfg, int64_t n, int32_t p_max, int32_t q_max, ClassLimits lim,
                                                          int bins, PlanHeader *h)
{
    __shared__ int32_t local[kPlanBins];
    __shared__ int32_t several;
    const int tid = static_cast<int>(threadIdx.x);
    for (int k = tid; k < bins; k += kPlanThreads) local[k] = 0;
    if (tid == 0) several = 0;
    __syncthreads();
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kPlanThreads + tid;
    if (i < n) {
        atomicAdd(&local[plan_bucket<T>(cfg, i, p_max, q_max, lim)], 1);
        if (!lim.by_work && cfg.q_req[i] > 1) several = 1;            // the same value whoever writes
    }
    __syncthreads();
    if (tid == 0 && several != 0) h->several = 1;
    for (int k = tid; k < bins; k += kPlanThreads)
        if (local[k] != 0) atomicAdd(&h->place[k], local[k]);
}

// One wavefront turns the counts of the first n_classes classes into places (the class after kClasses is the retry list of
// bi-greedy otherwise, which starts empty at position 0 of an array of its own).
__global__ __launch_bounds__(kWave) void plan_scan(PlanHeader *h, int giant_log2, int giant_log2_large, int n_classes)
{
    __shared__ int32_t before[kPlanBins + 1];
    const int lane = lane_id(), bins = n_classes * kWorkBuckets;
    int32_t run = 0;
    for (int at = 0; at < bins; at += kWave) {
        const int k = at + lane;
        const int32_t n = k < bins ? h->place[k] : 0, upto = run + wave_inclusive_scan(n);
        if (k < bins) { h->place[k] = upto - n; before[k] = upto - n; }
        run = __shfl(upto, kWave - 1, kWave);
    }
    if (lane == 0) before[bins] = run;
    __syncthreads();
    if (lane < n_classes) {
        h->class_begin[lane] = before[lane * kWorkBuckets];
        h->class_count[lane] = before[(lane + 1) * kWorkBuckets] - before[lane * kWorkBuckets];
    }
    if (lane == 0) h->large_left = kLargeClass < n_classes ? before[bins] - before[kLargeClass * kWorkBuckets] : 0;
    // buckets are ordered heaviest first: bucket b holds floor(log2) = kWorkBuckets - 1 - b
    const int last = (lane == 0 ? kClasses - 1 : kLargeClass + kClasses - 1), giants = kWorkBuckets - (lane == 0 ? giant_log2 : giant_log2_large);
    if (lane < 2 && last < n_classes && giants > 0)
        h->giant_count[lane] = before[last * kWorkBuckets + giants] - before[last * kWorkBuckets];
}

template <typename T>
__global__ __launch_bounds__(kPlanThreads) void plan_scatter(ConfigArrays cfg, int64_t n, int32_t p_max, int32_t q_max, ClassLimits lim,
                                                             int bins, PlanHeader *h, int32_t *order)
{
    __shared__ int32_t local[kPlanBins];                             // configurations of this block per bin, then the bin's first slot
    const int tid = static_cast<int>(threadIdx.x);
    for (int k = tid; k < bins; k += kPlanThreads) local[k] = 0;
    __syncthreads();
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kPlanThreads + tid;
    int b = 0, rank = 0;
    if (i < n) {
        b = plan_bucket<T>(cfg, i, p_max, q_max, lim);
        rank = atomicAdd(&local[b], 1);
    }
    __syncthreads();
    for (int k = tid; k < bins; k += kPlanThreads)
        if (local[k] != 0) local[k] = atomicAdd(&h->place[k], local[k]);
    __syncthreads();
    if (i < n) order[local[b] + rank] = static_cast<int32_t>(i);
}

// All four steps in one block for batches of up to kPlanSmall configurations: three launches less, each of which is waited for
// (960 machines, both port models: 249 -> 236 us in two calls).
// More than two rounds of the one block take longer than three launches (completion times of uni-greedy machines of 129 to 256 processors and one
// segment, us, four kernels and one block: 1000 51.7, 46.8; 2000 36.5, 34.8; 3000 36.9, 38.3; 4000 37.5, 41.3).
constexpr int kPlanSmallThreads = 1024, kPlanSmall = 2 * kPlanSmallThreads;
template <typename T>
__global__ __launch_bounds__(kPlanSmallThreads) void plan_small(ConfigArrays cfg, int n, int32_t p_max, int32_t q_max, ClassLimits lim, int n_classes,
                                                                PlanHeader *h, int32_t *order)
{
    __shared__ int32_t place[kPlanBins + 1];
    __shared__ int32_t several;
    const int tid = static_cast<int>(threadIdx.x), lane = lane_id(), bins = n_classes * kWorkBuckets;
    for (int k = tid; k <= kPlanBins; k += kPlanSmallThreads) place[k] = 0;
    if (tid == 0) several = 0;
    __syncthreads();
    int b[kPlanSmall / kPlanSmallThreads];
#pragma unroll
    for (int u = 0; u < kPlanSmall / kPlanSmallThreads; ++u) {
        const int i = tid + u * kPlanSmallThreads;
        b[u] = 0;
        if (i < n) {
            b[u] = plan_bucket<T>(cfg, i, p_max, q_max, lim);
            atomicAdd(&place[b[u]], 1);
            if (!lim.by_work && cfg.q_req[i] > 1) several = 1;
        }
    }
    __syncthreads();
    if (tid < kWave) {                                                   // counts into places, the end of the last bin behind them
        int32_t run = 0;
        for (int at = 0; at < bins; at += kWave) {
            const int k = at + lane;
            const int32_t c = k < bins ? place[k] : 0, upto = run + wave_inclusive_scan(c);
            if (k < bins) place[k] = upto - c;
            run = __shfl(upto, kWave - 1, kWave);
        }
        if (lane == 0) place[bins] = run;
    }
    __syncthreads();
    if (tid < kPlanClasses) {
        const bool used = tid < n_classes;
        const int32_t first = used ? place[tid * kWorkBuckets] : 0;
        h->ticket[tid] = 0ULL;
        h->class_begin[tid] = first;
        h->class_count[tid] = used ? place[(tid + 1) * kWorkBuckets] - first : 0;
    }
    if (tid < 2) {
        const int last = tid == 0 ? kClasses - 1 : kLargeClass + kClasses - 1, giants = kWorkBuckets - lim.giant_log2[tid];
        h->ticket_giant[tid] = 0ULL;
        h->giant_count[tid] = last < n_classes && giants > 0 ? place[last * kWorkBuckets + giants] - place[last * kWorkBuckets] : 0;
    }
    if (tid == 0) {
        h->large_left = kLargeClass < n_classes ? place[bins] - place[kLargeClass * kWorkBuckets] : 0;
        h->several = several;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPlanSmall / kPlanSmallThreads; ++u) {
        const int i = tid + u * kPlanSmallThreads;
        if (i < n) order[atomicAdd(&place[b[u]], 1)] = i;
    }
}

template <typename T> static void launch_plan_as(const PlanLaunch &L)
{
    const unsigned blocks = static_cast<unsigned>((L.n + kPlanThreads - 1) / kPlanThreads);
    const ClassLimits &lim = L.limits;
    const int classes = !lim.by_work ? kClasses : lim.large_p > 0 ? kPlanClasses : lim.wide_p > 0 ? kWideClass + 1 : kClasses;
    if (L.n <= kPlanSmall) {
        hipLaunchKernelGGL((plan_small<T>), dim3(1), dim3(kPlanSmallThreads), 0, L.stream, L.cfg, static_cast<int>(L.n), L.p_max, L.q_max, lim, classes,
                           L.header, L.order);
        return;
    }
    hipLaunchKernelGGL(plan_clear, dim3(1), dim3(256), 0, L.stream, L.header);
    hipLaunchKernelGGL((plan_hist<T>), dim3(blocks), dim3(kPlanThreads), 0, L.stream, L.cfg, L.n, L.p_max, L.q_max, lim, classes * kWorkBuckets, L.header);
    hipLaunchKernelGGL(plan_scan, dim3(1), dim3(kWave), 0, L.stream, L.header, lim.giant_log2[0], lim.giant_log2[1], classes);
    hipLaunchKernelGGL((plan_scatter<T>), dim3(blocks), dim3(kPlanThreads), 0, L.stream, L.cfg, L.n, L.p_max, L.q_max, lim, classes * kWorkBuckets, L.header, L.order);
}

hipError_t launch_plan(const PlanLaunch &L)
{
    if (L.cost == PRS_COST_I64) launch_plan_as<int64_t>(L); else launch_plan_as<double>(L);
    return hipGetLastError();
}

}  // namespace prs
