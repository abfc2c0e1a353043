// Uni-greedy schedules of machines of up to 1024 processors: the launch of their own (prs_uni_list.h has the lists).
#include "prs_uni_list.h"

namespace prs {

size_t uni_list_lds_bytes(int32_t procs) { return static_cast<size_t>(ListLds::bytes(procs)); }

// Segment numbers, runs of p - 1 equal ones, by whole wavefronts.  A wavefront takes several machines at a time, looked up by a lane
// each.
template <typename T>
__device__ __forceinline__ void list_segments(const ConfigArrays &cfg, int64_t n, int32_t p_max, int32_t q_max, const SchedOut &sched,
                                              unsigned long long *tickets)
{
    if (!sched.seg) return;
    const int lane = lane_id();
    // Long ones are left to the wavefronts that come first (a machine more or less is as long as a ticket takes); short ones are shared
    // out beforehand, without tickets.
    const bool shared = sched.pair_capacity / gridDim.x <= 65536;
    const int64_t share = shared ? (n + gridDim.x - 1) / gridDim.x : n / (static_cast<int64_t>(gridDim.x) * 4), most = shared ? kWave : 16;
    const int take = share < 1 ? 1 : static_cast<int>(share > most ? most : share);
    for (int64_t round = blockIdx.x;; round += gridDim.x) {
        const int64_t from = (shared ? round : next_ticket(tickets)) * take;
        if (from >= n) break;
        int64_t base = 0;
        int32_t procs = 0, segments = 0;
        if (lane < take && from + lane < n) {
            const Config<T> c = decode_config<T>(cfg, from + lane, p_max, q_max);
            base = sched.pair_offset[from + lane];
            if (c.status == PRS_CFG_OK && c.p <= kUniListProcs && base >= 0 && base + static_cast<int64_t>(c.p - 1) * c.q <= sched.pair_capacity) {
                procs = c.p; segments = c.q;
            }
        }
        // the shortest by their lanes
        const int few = (procs - 1) * segments;
        if (few > 0 && few <= kFewL) {
            int32_t *const out = sched.seg + base;
            int s = 0, r = 0;
            for (int j = 0; j < few; j += 4) {
                ListRow v;
#pragma unroll
                for (int b = 0; b < 4; ++b) { v[b] = static_cast<uint32_t>(s); const bool wrap = ++r == procs - 1; s += wrap ? 1 : 0; r = wrap ? 0 : r; }
                if (j + 4 <= few) {
                    *reinterpret_cast<ListRow *>(out + j) = v;
                } else {
#pragma unroll
                    for (int b = 0; b < 3; ++b)
                        if (j + b < few) out[j + b] = static_cast<int32_t>(v[b]);
                }
            }
            procs = 0;
        }
        for (int i = 0; i < take; ++i) {
            const int n1 = __builtin_amdgcn_readlane(procs, i) - 1, pairs = n1 * __builtin_amdgcn_readlane(segments, i);    // below 2^30
            if (n1 < 0) continue;
            const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(base)), i)),
                           hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(static_cast<uint64_t>(base) >> 32)), i));
            int32_t *const out = sched.seg + static_cast<int64_t>(static_cast<uint64_t>(hi) << 32 | lo);
            constexpr int step = 4 * kWave;
            int s = 4 * lane / n1, r = 4 * lane - s * n1;
            const int ds = step / n1, dr = step - ds * n1;
            for (int j = 4 * lane; j < pairs; j += step) {
                ListRow v;
                int sv = s, rv = r;
#pragma unroll
                for (int b = 0; b < 4; ++b) { v[b] = static_cast<uint32_t>(sv); const bool wrap = ++rv == n1; sv += wrap ? 1 : 0; rv = wrap ? 0 : rv; }
                if (j + 4 <= pairs) {
                    *reinterpret_cast<ListRow *>(out + j) = v;
                } else {
#pragma unroll
                    for (int b = 0; b < 3; ++b)
                        if (j + b < pairs) out[j + b] = static_cast<int32_t>(v[b]);
                }
                s += ds; r += dr;
                if (r >= n1) { r -= n1; ++s; }
            }
        }
    }
}

// One launch for the whole batch, and then the segment numbers.
template <typename T>
__global__ __launch_bounds__(kWave) void uni_list_kernel(ConfigArrays cfg, int64_t n, int32_t p_max, int32_t q_max, SchedOut sched,
                                                         PlanHeader *plan, const int32_t *order, int32_t procs)
{
    // behind wavefronts that have begun with them (uni_sched_kernel)
    bool begun = false;
    for (int k = kLargeClass; p_max > kUniListProcs && k < kPlanClasses; ++k) begun = begun || plan->class_count[k] != 0;
    uni_list_all<T>(procs, cfg, n, p_max, q_max, sched, plan, order, begun, false);
    list_segments<T>(cfg, n, p_max, q_max, sched, &plan->ticket_giant[0]);
}

hipError_t launch_uni_list(const UniLaunch &L)
{
    if (L.cost == PRS_COST_I64)
        hipLaunchKernelGGL((uni_list_kernel<int64_t>), dim3(L.grid), dim3(kWave), L.lds_bytes, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.sched,
                           L.plan, L.order, L.slot_p);
    else
        hipLaunchKernelGGL((uni_list_kernel<double>), dim3(L.grid), dim3(kWave), L.lds_bytes, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.sched,
                           L.plan, L.order, L.slot_p);
    return hipGetLastError();
}

}  // namespace prs
