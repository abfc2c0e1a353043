// greedy_schedule_batch for uni-greedy machines of up to 1024 processors on the CPU: the entry point, the plan's rule and the kernel are
// the library's own sources; launches run on emulated wavefronts.
#include <hip/hip_runtime.h>

#define launch_plan launch_plan_on_the_device
#include "../../paper_1310_4645_amd/csrc/prs_plan.hip"
#undef launch_plan
#include "../../paper_1310_4645_amd/csrc/prs_uni_list.hip"

namespace prs {

// the plan in one go: classes by the library's rule, heaviest bucket first
template <typename T> static void plan_as(const PlanLaunch &L)
{
    memset(L.header, 0, sizeof(PlanHeader));
    std::vector<std::vector<int32_t>> bins(kPlanClasses * kWorkBuckets);
    for (int64_t i = 0; i < L.n; ++i) bins[plan_bucket<T>(L.cfg, i, L.p_max, L.q_max, L.limits)].push_back(static_cast<int32_t>(i));
    int32_t at = 0;
    for (int c = 0; c < kPlanClasses; ++c) {
        L.header->class_begin[c] = at;
        for (int b = 0; b < kWorkBuckets; ++b)
            for (int32_t i : bins[c * kWorkBuckets + b]) L.order[at++] = i;
        L.header->class_count[c] = at - L.header->class_begin[c];
    }
}
hipError_t launch_plan(const PlanLaunch &L)
{
    if (L.cost == PRS_COST_I64) plan_as<int64_t>(L); else plan_as<double>(L);
    return hipSuccess;
}

// In place of the launch of large machines, of which there are none: what its idle wavefronts do, as long as a large one
// would not be done (help_for operations, 0: no such launch).
static int64_t help_for;
template <typename T>
__global__ void help_kernel(ConfigArrays cfg, int64_t n, int32_t p_max, int32_t q_max, SchedOut sched, PlanHeader *plan, const int32_t *order, int32_t procs)
{
    uni_list_all<T>(procs, cfg, n, p_max, q_max, sched, plan, order, true, true);
}
hipError_t launch_uni_sched(const UniLaunch &L)
{
    if (help_for == 0) return hipSuccess;
    L.plan->class_count[kLargeClass] = 1;
    L.plan->large_left = 1;
    emu::clear = &L.plan->large_left;
    emu::clear_at = help_for;
    if (L.cost == PRS_COST_I64)
        hipLaunchKernelGGL((help_kernel<int64_t>), dim3(2), dim3(kWave), L.lds_bytes, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.sched, L.plan, L.order, L.list_procs);
    else
        hipLaunchKernelGGL((help_kernel<double>), dim3(2), dim3(kWave), L.lds_bytes, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.sched, L.plan, L.order, L.list_procs);
    emu::clear = nullptr;
    return hipSuccess;
}

// not reached: everything but uni-greedy schedules of small machines
#define PRS_NOT_HERE(what) { emu::fault(what, 0, 0); return 1; }
hipError_t launch_uni_times(const UniLaunch &) PRS_NOT_HERE("uni_times")
hipError_t launch_uni_wide(const UniLaunch &) PRS_NOT_HERE("uni_wide")
hipError_t launch_bi(const BiLaunch &) PRS_NOT_HERE("bi")
hipError_t launch_bi_block(const BiLaunch &) PRS_NOT_HERE("bi_block")
hipError_t launch_bi_group(const BiGroupLaunch &) PRS_NOT_HERE("bi_group")
hipError_t launch_replay(const ReplayLaunch &) PRS_NOT_HERE("replay")
hipError_t launch_threshold(const ThresholdLaunch &) PRS_NOT_HERE("threshold")
hipError_t launch_alu_ceiling(int64_t, int32_t, double *, hipStream_t) PRS_NOT_HERE("alu")
hipError_t replay_static_scratch(void **) PRS_NOT_HERE("replay")
size_t replay_workspace_bytes(int32_t, int32_t) { return 0; }
size_t replay_scratch_bytes(int32_t, int32_t) { return 0; }
size_t uni_times_lds_bytes(int32_t, bool) { return 1024; }
int32_t uni_times_slot_runs(int32_t) { return 0; }
size_t uni_times_slot_bytes(int32_t, bool) { return 0; }
size_t uni_sched_lds_bytes() { return 40960; }
size_t uni_sched_slot_bytes(int32_t) { return 0; }
size_t uni_wide_slot_bytes(int32_t) { return 0; }
size_t uni_wide_lds_bytes() { return 0; }
size_t bi_small_bytes(int32_t, int32_t) { return 0; }
size_t bi_bitmap_bytes(int32_t, int32_t) { return 0; }
size_t bi_masks_bytes(int32_t) { return 0; }
size_t bi_slot_bytes(int32_t, int32_t, bool) { return 0; }
size_t bi_group_lds_bytes(int) { return 1024; }
int bi_group_list_capacity(int) { return 0; }
size_t bi_block_slot_bytes(int32_t, int32_t) { return 0; }
size_t bi_block_lds_bytes(int32_t) { return 0; }

}  // namespace prs

#include "../../paper_1310_4645_amd/csrc/prs_api.hip"

extern "C" {
// types: report bytes of LDS used as two types;
// limit: operations between lanes a call may take; poke: after poke_at of them (0: never) so many bytes of LDS are overwritten
void emu_begin(int types, int64_t limit, int backwards, int64_t poke_at, int64_t poke_place, int64_t poke_value, int64_t poke_size)
{
    emu::types = types != 0; emu::waits = 0; emu::wait_limit = limit; emu::backwards = backwards != 0; emu::faults = 0; emu::first_fault[0] = 0; emu::stopped = false;
    emu::poke_at = poke_at; emu::poke_place = poke_place; emu::poke_value = poke_value; emu::poke_size = poke_size;
}
void emu_help(int64_t operations) { prs::help_for = operations; }
int64_t emu_waits() { return emu::waits; }
int emu_stopped() { return emu::stopped; }
int emu_faults() { return emu::faults; }
const char *emu_first_fault() { return emu::first_fault; }
}
