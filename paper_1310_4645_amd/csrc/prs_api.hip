// C ABI of the library (declared in include/prs.h): argument checks, workspace
// carving and kernel launches.  No device memory is allocated here.
#include "prs_device.h"
#include "prs_launch.h"

#include <algorithm>

namespace prs {

constexpr size_t kHeaderBytes = 256;
constexpr size_t kMaxWorkspace = static_cast<size_t>(16) << 30;   // slots of the global-memory class, at most (if 256 of them fit)

__global__ void clear_words(unsigned long long *w, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) w[i] = 0ULL;
}

hipError_t launch_clear(unsigned long long *words, int count, hipStream_t stream)
{
    hipLaunchKernelGGL(clear_words, dim3((count + 63) / 64), dim3(64), 0, stream, words, count);
    return hipGetLastError();
}

// pair_offset[i] = sum_{j<i} (p_j - 1) q_eff_j; one block, sequential carry over tiles of 1024.
template <typename T>
__global__ __launch_bounds__(1024) void offsets_kernel(ConfigArrays cfg, int64_t n, int32_t p_max, int32_t q_max,
                                                       int64_t *pair_offset)
{
    __shared__ int64_t s_wave[16];
    __shared__ int64_t s_carry;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) { s_carry = 0; pair_offset[0] = 0; }
    __syncthreads();
    for (int64_t base = 0; base < n; base += 1024) {
        const int64_t i = base + tid;
        int64_t cnt = 0;
        if (i < n) {
            const Config<T> c = decode_config<T>(cfg, i, p_max, q_max);
            if (c.status == PRS_CFG_OK) cnt = static_cast<int64_t>(c.p - 1) * c.q;
        }
        int64_t inc = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up(inc, o, 64);
            if (lane >= o) inc += u;
        }
        if (lane == 63) s_wave[wv] = inc;
        __syncthreads();
        int64_t before = s_carry;
        for (int w = 0; w < wv; ++w) before += s_wave[w];
        if (i < n) pair_offset[i + 1] = before + inc;
        __syncthreads();
        if (tid == 1023) s_carry = before + inc;
        __syncthreads();
    }
}

hipError_t launch_offsets(const OffsetsLaunch &L)
{
    if (L.cost == PRS_COST_I64)
        hipLaunchKernelGGL((offsets_kernel<int64_t>), dim3(1), dim3(1024), 0, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.pair_offset);
    else
        hipLaunchKernelGGL((offsets_kernel<double>), dim3(1), dim3(1024), 0, L.stream, L.cfg, L.n, L.p_max, L.q_max, L.pair_offset);
    return hipGetLastError();
}

// ---- size classes and workspace layout (shared by prs_workspace_bytes and the launches) --------------
//
// A batch is split into classes, each run by the kernel and the LDS allocation that fit it:
//   uni-greedy times:                 by number of pairs; 1, 2, 4, 8, 16, 32 or 64 lanes per configuration in one launch, machines
//                                     of more than kUniSmallProcs processors in another;
//   uni-greedy schedules:             by processors and number of pairs; 1, 2, 4, 8, 16 or 32 lanes per configuration in one launch,
//                                     machines of more than kUniListProcs processors (1, 8, 16, 32 or 64 lanes) in another, whose
//                                     idle wavefronts begin with the first;
//   bi-greedy:                        1, 2, 4, 8 or 16 lanes per configuration for p <= 64 / 128 / 256 / 512 / 1024 and
//                                     q <= 1023; the general kernel for the rest and for reruns.
enum ClassKind { kUniTimes, kUniSched, kUniList, kBiGroup, kBiGeneral, kBiBlock, kUniWide };
constexpr size_t kLdsPerCU = 160 * 1024, kLdsPerBlockMax = 64 * 1024, kBitmapLdsMax = 24 * 1024;
constexpr int kCUs = 256, kSIMDs = 4 * kCUs, kMaxBlocksPerCU = 24, kGlobalClassGrid = 1024;
// LDS is given out in units of 1280 bytes: six one-wavefront blocks of 26,880 bytes run on a CU side by side, five of 27,300.
constexpr size_t kLdsUnit = 1280;
static int64_t blocks_per_cu(size_t lds_bytes)
{
    return static_cast<int64_t>(kLdsPerCU / ((lds_bytes + kLdsUnit - 1) / kLdsUnit * kLdsUnit));
}
constexpr int32_t kGroupQMax = 1023;   // the several-per-wavefront bi-greedy kernel counts sent segments in 10 bit planes
constexpr int kUniGroupSizes = 3;        // group sizes below the largest; the classes between them and the last stay empty
// completion times: a configuration gets 1, 2, 4, 8 or 16 lanes with at most so many pairs and processors, more get 32, and 64
// from 2^kUniTimesGiantLog2 pairs on.  With fewer lanes the deep ring of a group overflows and the configuration starts again
// in the workspace (limits twice as high: 300 of the 100,000, 4.65 ms against 4.15; without the limits on processors 80, 3.75
// against 3.55), with more of them lanes wait for their neighbours (limits half as high: 4.45 ms).  64 lanes halve the time of
// the longest configurations (4 million pairs: 31 ms on 32 lanes, 13 on 64).  Compositions have few segments and deeper rings: no
// limit on processors (1.46 ms against 1.6 to 2.8).
constexpr int64_t kUniTimesWork[kClasses - 1] = {256, 2048, 8192, 32768, 131072};
constexpr int32_t kUniTimesProcs[kClasses - 1] = {36, 64, 128, 320, INT32_MAX};
constexpr int kUniTimesGiantLog2 = 19;
constexpr int64_t kUniWorkSched[kUniGroupSizes] = {1024, 65536, 262144};  // schedules of large machines: by 1, 8, 16 lanes
constexpr int64_t kUniWorkList[kClasses - 1] = {512, 2048, 8192, 32768, 131072};   // schedules of the others: by 1, 2, 4, 8, 16 lanes
// uni-greedy completion times: machines of at least this many processors would get a block per configuration.  Off: on the
// large-machine sweep it is 2 to 3 times slower than the segment pipeline was pair by pair, and that one is now more than 50
// times faster; the kernel stays reachable through prs_tuning.
constexpr int32_t kUniWideProcs = INT32_MAX;

struct ClassSpec {
    ClassKind kind;
    int lpc;                  // kBiGroup: lanes per configuration
    size_t rows_per_group;    // kBiGroup: words of sent-bit rows per configuration slot
    int32_t p_cap;            // capacity of the per-processor arrays of this class
    int32_t q_cap;            // capacity of its per-segment arrays
    bool lds;                 // state (uni batch) / small arrays and maybe the bitmap (bi general) in LDS
    size_t lds_bytes;
    int32_t lds_bitmap_bytes;
    size_t slot_bytes, slot_offset;
    int grid;
    int slots = 0;            // kUniSched: blocks of the grid that have a slot; the others only run lists
};

struct Layout {
    size_t header, order, retry, total;
    ClassLimits limits;
    ClassSpec cls[kClasses];
    ClassSpec rerun;              // bi-greedy: the one-wavefront kernel for configurations the group kernel hands back
    ClassSpec wide;               // uni-greedy completion times: the block-per-configuration kernel (grid 0: not used)
    bool help;                    // completion times: wavefronts without a large machine begin with the small ones
    ClassSpec large;              // uni-greedy: machines of more than kUniSmallProcs processors (grid 0: none)
    bool bi_on[kClasses - 1];     // bi-greedy group classes a configuration can fall into
};

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// the one-configuration-per-wavefront bi-greedy kernel: where its arrays go for machines of up to p_cap processors
static void general_spec(ClassSpec &c, int32_t p_cap, int32_t q_cap)
{
    c.kind = kBiGeneral;
    c.p_cap = p_cap;
    c.q_cap = q_cap;
    c.lds = false; c.lds_bytes = 0; c.lds_bitmap_bytes = 0; c.lpc = 0; c.rows_per_group = 0;
    const size_t small = bi_small_bytes(p_cap, q_cap), bitmap = bi_bitmap_bytes(p_cap, q_cap);
    if (small <= kLdsPerBlockMax / 2) {
        c.lds = true;
        c.lds_bitmap_bytes = static_cast<int32_t>(bitmap < kBitmapLdsMax ? bitmap : kBitmapLdsMax);
        c.lds_bytes = small + static_cast<size_t>(c.lds_bitmap_bytes);
    } else if (bi_masks_bytes(p_cap) <= kLdsPerBlockMax) {
        c.lds_bytes = bi_masks_bytes(p_cap);             // bit sets in LDS, lists and counters in the slot
    }
    c.slot_bytes = bi_slot_bytes(p_cap, q_cap, c.lds);
}

// Schedules of few segments: lanes beyond the segments have nothing to do (the first segment takes none), so what counts is how many
// lanes that have something to do fit a CU: with g lanes for the largest machine, groups and wavefronts that find room, of which
// more than seven only share cycles.  Machines of more than 16 processors are not run by one lane, and one segment alone goes no
// further than 20 processors a lane: the lanes of a group lay the first one down together.  100,000 equal machines, us, with 1, 2, 4, 8 and 16
// lanes: 31 processors and 2 segments 237, 150, 191, 271, -; 100 and 2 -, 532, 565, 761, 1372; 64 and 1 294, 174, 114, 119, 147; 481 and 2 of 8 and 16
// lanes 6340, 6998.  Four wavefronts at least if the segments are more than a few (20,000 of 480 and 8, 8 and 16 lanes: 5034, 4450).
constexpr int32_t kFewSegments = 16;
// Most wavefronts of the list kernel per CU: small machines find room for more, which only share cycles and have to be started (us with
// 10, 12 and 16: 20,000 machines of 5 processors and 30 segments 134, 136, 194; of 100 and 30 1459, 1277, 1459).
constexpr int32_t kListWavesPerCU = 12;
// Beside machines of more than 1024 processors (`large`) the lists also have to fit the LDS of their rings.
static int32_t few_segments_lane_p(int32_t p, int32_t q, bool large)
{
    int32_t best = kUniListLaneProcs;
    int64_t most = 0;
    for (int lanes = p <= 16 ? 1 : 2; lanes <= 32; lanes *= 2) {
        const int32_t room = std::max((p + lanes - 1) / lanes, 4);
        const int64_t waves = std::min<int64_t>(blocks_per_cu(uni_list_lds_bytes(room)), 7);
        if (room > (q == 1 ? 20 : 64) || (q > 4 && waves < 4) || (large && uni_list_lds_bytes(room) > uni_sched_lds_bytes())) continue;
        const int64_t busy = waves * (kWave / lanes) * std::min(lanes, std::max(q - 1, 1));
        if (busy > most) { most = busy; best = room; }
    }
    return best;
}

static Layout make_layout(int call, int model, int64_t n, int32_t p_max, int32_t q_max, const prs_tuning *tuning = nullptr,
                          bool compositions = false)
{
    Layout L;
    const bool sched = call == PRS_CALL_SCHEDULE;
    L.header = 0;
    L.order = plan_header_bytes();
    L.retry = L.order + align256(static_cast<size_t>(n < 1 ? 1 : n) * 4);
    size_t off = L.retry + align256(static_cast<size_t>(n < 1 ? 1 : n) * 4);
    // which configurations go where
    const int32_t plim[kClasses - 1] = {64, 128, 256, 512, 1024};
    for (int k = 0; k < kClasses - 1; ++k) L.limits.p[0][k] = L.limits.p[1][k] = plim[k];
    L.limits.q = kGroupQMax;
    L.limits.by_work = 0;
    L.limits.large_p = 0;
    for (int set = 0; set < 2; ++set) {
        for (int k = 0; k < kClasses - 1; ++k) L.limits.work[set][k] = 0;
        L.limits.giant_log2[set] = kGiantLog2;
        L.limits.lanes_log2[set] = 0;
    }
    L.limits.lane_p = 0;
    L.limits.wide_p = 0;
    L.large.grid = 0;
    L.help = false;
    L.wide.grid = 0; L.wide.slot_bytes = 0; L.wide.slot_offset = 0;
    static const int group_lpc[kClasses - 1] = {1, 2, 4, 8, 16};
    if (model == PRS_UNI) {
        // Classes by number of pairs (1, 2, 4, 8, 16 or 32 lanes per configuration), all run by one launch, described by class 0.
        // Machines with more than kUniSmallProcs processors take a launch of their own.  Completion times: its wavefronts have
        // larger rings: a bound p_max above the machines of a batch, or one large machine among them, does not cost the others
        // their wavefronts (100,000 machines of up to 1024 processors with p_max = 16384: 15.5 ms with the large rings for all,
        // one wavefront per CU).  Schedules: the lists of the others have their processors in LDS, those of the large ones lie in
        // the workspace (1, 8, 16 or 32 lanes per configuration).
        L.limits.by_work = 1;
        const bool has_large = p_max > kUniSmallProcs;
        if (has_large) L.limits.large_p = kUniSmallProcs;
        const int32_t p_small = has_large ? kUniSmallProcs : p_max;
        if (sched) {
            // Room for so many processors per lane: 16 lanes for the largest machine, the group size up to which most lanes of a
            // pipeline have something to do, but no more than lets six wavefronts share a CU.
            L.limits.lane_p = std::min(std::max((p_small + 15) / 16, 8), kUniListLaneProcs);
            if (q_max <= kFewSegments) L.limits.lane_p = few_segments_lane_p(p_small, q_max, has_large);
        }
        for (int set = 0; set < 2; ++set) {
            const bool lists = sched && set == 0, rings = sched && set == 1;
            int64_t *const work = L.limits.work[set];
            for (int k = 0; k < kClasses - 1; ++k) {
                L.limits.p[set][k] = sched || compositions ? INT32_MAX : kUniTimesProcs[k];
                work[k] = rings ? kUniWorkSched[k < kUniGroupSizes ? k : kUniGroupSizes - 1] : lists ? kUniWorkList[k] : kUniTimesWork[k];
            }
            if (!rings) {
                // A batch that leaves lanes without a configuration gives each of its configurations more of them.
                const size_t lds = lists ? uni_list_lds_bytes(L.limits.lane_p) : uni_times_lds_bytes(set ? p_max : p_small, compositions);
                const int64_t lanes = blocks_per_cu(lds) * kCUs * kWave;
                for (int k = 0; k < kClasses - 1; ++k)
                    if (n << (k + 1) <= lanes) work[k] = 0;
                if (!lists) L.limits.giant_log2[set] = kUniTimesGiantLog2;
                if (!lists && n << 6 <= lanes) L.limits.giant_log2[set] = 0;
                else L.limits.lanes_log2[set] = 1;
            } else {
                // The same for schedules of large machines: 64, 32, 16 or 8 lanes where the batch leaves that many idle.
                const int64_t lanes = blocks_per_cu(uni_sched_lds_bytes()) * kCUs * kWave;
                static const int more[kUniGroupSizes] = {3, 4, 5};            // the next group size: 8, 16, 32 lanes
                for (int k = 0; k < kClasses - 1; ++k)
                    if (n << more[k < kUniGroupSizes ? k : kUniGroupSizes - 1] <= lanes) work[k] = 0;
                if (n << 6 <= lanes) L.limits.giant_log2[set] = 0;
            }
            if (tuning) {                                              // never changes a result, only who runs what
                L.limits.lanes_log2[set] = 0;
                L.limits.giant_log2[set] = sched ? kGiantLog2 : kUniTimesGiantLog2;
                for (int k = 0; k < kClasses - 1; ++k) L.limits.p[set][k] = INT32_MAX;
                const int64_t a = tuning->uni_group_pairs[0], b = tuning->uni_group_pairs[1], c3 = tuning->uni_group_pairs[2];
                if (a >= 0 && b >= a && c3 >= b) {
                    if (rings) {
                        work[0] = a; work[1] = b;
                        for (int k = 2; k < kClasses - 1; ++k) work[k] = c3;
                    } else {                                           // 1, 4 and 16 lanes; nothing for 2 and 8
                        work[0] = work[1] = a;
                        work[2] = work[3] = b;
                        work[4] = c3;
                    }
                }
                if (tuning->uni_wave_log2 > 0 && tuning->uni_wave_log2 < kWorkBuckets) L.limits.giant_log2[set] = tuning->uni_wave_log2;
            }
        }
        auto uni_spec = [&](ClassSpec &c, int32_t p) {                 // one launch for machines of up to p processors
            c.q_cap = q_max;
            c.lpc = 0; c.rows_per_group = 0; c.lds = true; c.lds_bitmap_bytes = 0;
            if (sched && p <= kUniListProcs) {                         // everything in LDS
                c.kind = kUniList;
                c.p_cap = L.limits.lane_p; c.lds_bytes = uni_list_lds_bytes(c.p_cap); c.slot_bytes = 0;
            } else if (sched) {
                c.kind = kUniSched;
                c.p_cap = (p + 15) / 16 * 16;                          // keeps every per-lane array 64-byte aligned
                c.lds_bytes = uni_sched_lds_bytes(); c.slot_bytes = uni_sched_slot_bytes(c.p_cap);
            } else {
                c.kind = kUniTimes;
                c.p_cap = uni_times_slot_runs(p);                      // runs of a lane's ring
                c.lds_bytes = uni_times_lds_bytes(p, compositions);
                c.slot_bytes = uni_times_slot_bytes(c.p_cap, compositions || p > kUniSmallProcs);
            }
            int64_t g = blocks_per_cu(c.lds_bytes) * kCUs;
            if (c.kind == kUniList && g > kListWavesPerCU * kCUs) g = kListWavesPerCU * kCUs;
            if (c.kind != kUniSched && g > n) g = n < 1 ? 1 : n;
            size_t bytes = static_cast<size_t>(g) * c.slot_bytes;
            if (sched) {
                while (g > 1 && static_cast<size_t>(g) * c.slot_bytes > kMaxWorkspace) g /= 2;
                bytes = static_cast<size_t>(g) * c.slot_bytes;
            } else if (bytes > kMaxWorkspace) {
                bytes = kMaxWorkspace;
                g = static_cast<int64_t>(bytes / c.slot_bytes);
            }
            c.grid = c.slots = static_cast<int>(g);
            if (c.kind == kUniSched) c.grid = static_cast<int>(blocks_per_cu(c.lds_bytes) * kCUs);
            c.slot_offset = off;
            return align256(bytes);
        };
        size_t slots = uni_spec(L.cls[0], p_small);
        for (int k = 1; k < kClasses; ++k) { L.cls[k] = L.cls[0]; L.cls[k].grid = 0; L.cls[k].slot_bytes = 0; }
        if (has_large) {                                               // the launches follow each other and share the slots
            // Completion times: a batch whose small machines leave lanes idle is bound by its longest chains: these begin beside the large
            // machines (3000 machines, 81 of them of 1024 to 20000 processors: 5.9 -> 4.0 ms).  A larger one is bound by how many
            // run at once, which is one wavefront per CU there and five in the launch that follows (30000 machines: 5.9 -> 6.4).
            // Schedules: four and six wavefronts, so they always do (uni_sched_kernel).
            L.help = !sched && n << 4 <= blocks_per_cu(uni_times_lds_bytes(p_small, compositions)) * kCUs * kWave;
            if (!sched && p_max > kUniMidProcs) slots = std::max(slots, uni_spec(L.large, kUniMidProcs));   // more wavefronts: no less than for that bound
            slots = std::max(slots, uni_spec(L.large, p_max));
        }
        // completion times of machines with thousands of processors: a block per configuration
        if (!sched) {
            int32_t wide_p = kUniWideProcs;
            if (tuning && tuning->uni_wide_procs > 0) wide_p = tuning->uni_wide_procs;
            if (p_max >= wide_p) L.limits.wide_p = wide_p;
            {                                                          // runs before the others, in the same slots (smaller than theirs)
                ClassSpec &c = L.wide;
                c.kind = kUniWide; c.p_cap = p_max; c.q_cap = q_max; c.lds = true; c.lds_bytes = uni_wide_lds_bytes();
                c.lds_bitmap_bytes = 0; c.lpc = 0; c.rows_per_group = 0;
                c.slot_bytes = uni_wide_slot_bytes(p_max);
                int64_t g = 2 * kCUs;
                while (g > 1 && static_cast<size_t>(g) * c.slot_bytes > (static_cast<size_t>(1) << 30)) g /= 2;   // at most 1 GiB of the workspace
                if (g > n) g = n < 1 ? 1 : n;
                c.grid = static_cast<int>(g);
                c.slot_offset = off;
                slots = std::max(slots, align256(static_cast<size_t>(c.grid) * c.slot_bytes));
            }
        }
        off += slots;
        L.total = off;
        return L;
    }
    for (int k = 0; k < kClasses; ++k) {
        ClassSpec &c = L.cls[k];
        const bool last = k == kClasses - 1;
        c.p_cap = last ? p_max : (L.limits.p[0][k] < p_max ? L.limits.p[0][k] : p_max);
        c.q_cap = q_max;
        c.lds = false; c.lds_bytes = 0; c.lds_bitmap_bytes = 0; c.slot_bytes = 0; c.lpc = 0; c.rows_per_group = 0;
        const bool possible = last || k == 0 || L.limits.p[0][k - 1] < p_max;   // can a configuration land here?
        if (!last) {
            // several configurations per wavefront; the slot of a wavefront holds the sent-bit rows of its groups
            c.kind = kBiGroup;
            c.lpc = group_lpc[k];
            c.lds = true;
            c.lds_bytes = bi_group_lds_bytes(c.lpc);
            const int32_t q_cap = q_max < kGroupQMax ? q_max : kGroupQMax;
            c.rows_per_group = static_cast<size_t>(q_cap) * c.lpc;
            c.slot_bytes = c.rows_per_group * 8 * (64 / c.lpc);
        } else if (p_max > L.limits.p[0][kClasses - 2] && bi_block_lds_bytes(c.p_cap) <= kLdsPerBlockMax) {
            // thousands of processors: one block of 8 wavefronts per configuration
            c.kind = kBiBlock;
            c.lds_bytes = bi_block_lds_bytes(c.p_cap);
            c.slot_bytes = bi_block_slot_bytes(c.p_cap, q_max);
        } else {
            // one configuration per wavefront: many segments on a small machine, or more processors than the block
            // kernel's LDS holds
            general_spec(c, c.p_cap, q_max);
        }
        int64_t g;
        if (c.kind == kBiBlock) {
            g = 2 * kCUs;
        } else if (c.lds) {
            int64_t per_cu = static_cast<int64_t>(kLdsPerCU / (c.lds_bytes < 1024 ? 1024 : c.lds_bytes));
            if (per_cu > kMaxBlocksPerCU) per_cu = kMaxBlocksPerCU;
            if (per_cu < 1) per_cu = 1;
            g = per_cu * kCUs;
        } else {
            g = kGlobalClassGrid;
        }
        while (g > 256 && static_cast<size_t>(g) * c.slot_bytes > kMaxWorkspace) g /= 2;   // big slots: fewer resident blocks
        if (g > n) g = n < 1 ? 1 : n;
        if (!possible) g = 0;
        c.grid = static_cast<int>(g);
        if (!last) L.bi_on[k] = possible;
    }
    // the group classes share one resident set of blocks, carried by class 0: as many as the largest LDS
    // allocation of a usable class allows (their slots of sent-bit rows have the same size)
    {
        int g = 0;
        for (int k = 0; k < kClasses - 1; ++k)
            if (L.bi_on[k] && (g == 0 || L.cls[k].grid < g)) g = L.cls[k].grid;
        for (int k = 0; k < kClasses - 1; ++k) L.cls[k].grid = k == 0 ? g : 0;
    }
    for (int k = 0; k < kClasses; ++k) {
        ClassSpec &c = L.cls[k];
        c.slot_offset = off;
        off += align256(static_cast<size_t>(c.grid) * c.slot_bytes);
    }
    // reruns come from the group classes only: at most 1024 processors and 1023 segments
    {
        ClassSpec &c = L.rerun;
        general_spec(c, p_max < L.limits.p[0][kClasses - 2] ? p_max : L.limits.p[0][kClasses - 2], q_max < kGroupQMax ? q_max : kGroupQMax);
        int64_t g = kGlobalClassGrid;
        if (c.lds) {
            int64_t per_cu = static_cast<int64_t>(kLdsPerCU / (c.lds_bytes < 1024 ? 1024 : c.lds_bytes));
            if (per_cu > kMaxBlocksPerCU) per_cu = kMaxBlocksPerCU;
            if (per_cu < 1) per_cu = 1;
            g = per_cu * kCUs;
        }
        if (g > n) g = n < 1 ? 1 : n;
        c.grid = static_cast<int>(g);
        c.slot_offset = off;
        off += align256(static_cast<size_t>(c.grid) * c.slot_bytes);
    }
    L.total = off;
    return L;
}

static bool bad_common(const prs_configs *cfg, int64_t n, int model, int cost, int32_t p_max, int32_t q_max)
{
    if (!cfg || n < 0 || n >= (INT64_C(1) << 31) || (model != PRS_UNI && model != PRS_BI) ||
        (cost != PRS_COST_I64 && cost != PRS_COST_F64))
        return true;
    if (p_max < 2 || p_max > (1 << 20) || q_max < 1 || q_max > (1 << 20)) return true;
    if (n > 0 && (!cfg->p || !cfg->q_req || !cfg->m || !cfg->alpha || !cfg->beta || !cfg->gamma)) return true;
    return false;
}

static int run_greedy(int call, const prs_configs *cfg, int64_t n, int model, int cost, int32_t p_max, int32_t q_max,
                      const TimesOut &times, const SchedOut &sched, void *workspace, size_t workspace_bytes, void *stream,
                      const prs_tuning *tuning, int32_t comp_m = 0)
{
    if (comp_m > 0 && (call != PRS_CALL_SIMULATE || model != PRS_UNI)) return PRS_EINVAL;   // compositions: uni-greedy times only
    if (n == 0) return PRS_OK;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return PRS_EINVAL;
    const Layout lay = make_layout(call, model, n, p_max, q_max, tuning, comp_m > 0);
    if (workspace_bytes < lay.total) return PRS_ENOSPC;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    PlanLaunch P;
    P.cfg = ConfigArrays{cfg->p, cfg->q_req, cfg->m, cfg->alpha, cfg->beta, cfg->gamma};
    P.cfg.comp_m = comp_m;
    P.n = n; P.p_max = p_max; P.q_max = q_max; P.cost = cost;
    P.limits = lay.limits;
    P.header = reinterpret_cast<PlanHeader *>(ws + lay.header);
    P.order = reinterpret_cast<int32_t *>(ws + lay.order);
    P.stream = st;
    if (launch_plan(P) != hipSuccess) return PRS_EDEVICE;
    int32_t *retry = reinterpret_cast<int32_t *>(ws + lay.retry);
    auto general = [&](const ClassSpec &c, const int32_t *order, int cls) {          // batch / general kernels
        UniLaunch L;
        L.cfg = P.cfg; L.n = n;
        L.p_max = p_max; L.q_max = q_max; L.model = model; L.cost = cost;
        L.want_schedule = call == PRS_CALL_SCHEDULE;
        L.times = times; L.sched = sched;
        L.plan = P.header; L.order = order; L.cls = cls; L.help = lay.help;
        L.list_entries = (tuning && tuning->bi_list_entries > 0 && tuning->bi_list_entries < kWave) ? tuning->bi_list_entries : kWave;
        L.lds_p = c.lds ? c.p_cap : 0;
        L.lds_bitmap_bytes = c.lds_bitmap_bytes;
        L.lds_bytes = c.lds_bytes;
        L.slots = ws + c.slot_offset;
        L.slot_bytes = c.slot_bytes;
        L.slot_p = c.p_cap; L.slot_q = c.q_cap;
        L.grid = c.grid;
        L.stream = st;
        if (c.kind == kUniTimes) return launch_uni_times(L);
        if (c.kind == kUniList) return launch_uni_list(L);
        L.slot_count = c.slots; L.list_procs = lay.limits.lane_p;
        if (c.kind == kUniSched) return launch_uni_sched(L);
        if (c.kind == kBiBlock) return launch_bi_block(L);
        if (c.kind == kUniWide) return launch_uni_wide(L);
        return launch_bi(L);
    };
    // the class with the longest-running configurations first; a class without configurations ends at once
    if (lay.limits.wide_p > 0 && general(lay.wide, P.order, kWideClass) != hipSuccess) return PRS_EDEVICE;
    if (lay.large.grid > 0 && general(lay.large, P.order, kLargeClass) != hipSuccess) return PRS_EDEVICE;
    bool groups_done = false;
    for (int k = kClasses - 1; k >= 0; --k) {
        const ClassSpec &c = lay.cls[k];
        if (c.grid == 0) continue;                       // no configuration can fall in this class
        if (c.kind == kBiGroup) {
            if (groups_done) continue;                   // the group sizes share one launch
            groups_done = true;
            BiGroupLaunch G;
            G.cfg = P.cfg; G.p_max = p_max; G.q_max = q_max; G.model = model; G.cost = cost;
            G.want_schedule = call == PRS_CALL_SCHEDULE;
            G.times = times; G.sched = sched; G.plan = P.header; G.order = P.order;
            G.retry = retry;
            // one resident set of blocks (class 0 carries its size and the sent-bit rows), split between the
            // classes the blocks start with
            const ClassSpec &c0 = lay.cls[0];
            int total = c0.grid, enabled = 0;
            static const int share[kBiGroupSizes] = {2, 2, 3, 6, 7};      // twentieths of the blocks that start with class 0 .. 4 (measured; flat around these)
            for (int g = 0; g < kBiGroupSizes; ++g) {
                G.parts.on[g] = lay.cls[g].kind == kBiGroup && lay.cls[g].lpc > 0 && lay.cls[g].rows_per_group > 0 && lay.bi_on[g];
                G.parts.rows_per_group[g] = lay.cls[g].rows_per_group;
                const int cap = bi_group_list_capacity(lay.cls[g].lpc > 0 ? lay.cls[g].lpc : 1);
                G.parts.list_entries[g] = (tuning && tuning->bi_list_entries > 0 && tuning->bi_list_entries < cap) ? tuning->bi_list_entries : cap;
                if (G.parts.on[g]) enabled += share[g];
            }
            int given = 0;
            for (int g = kBiGroupSizes - 1; g >= 0; --g) {
                G.parts.start[g] = G.parts.on[g] ? total * share[g] / enabled : 0;
                given += G.parts.start[g];
            }
            for (int g = kBiGroupSizes - 1; g >= 0; --g)
                if (G.parts.on[g]) { G.parts.start[g] += total - given; break; }   // rounding remainder
            G.parts.rows = reinterpret_cast<uint64_t *>(ws + c0.slot_offset);
            G.parts.rows_per_block = c0.slot_bytes / 8;
            // Configurations that share a wavefront wait for each other's paths: a batch that leaves wavefronts without one
            // spreads out, unless all of it are single segments (960 machines of 2 to 16 processors, both port models: 488 ->
            // 255 us; 500 machines of 2 to 1024 processors and up to 512 segments 18.5 -> 10.7 ms, of 2 to 64 processors
            // 16.8 -> 7.1; 500 equal ones of 1024 and 512 10.4 -> 11.5, of 40 and 8 with schedules 1.25 -> 0.52).
            // With 64 or 32 groups to a wavefront that ends at one wavefront per SIMD, more only share its cycles (20,000
            // machines of 60 to 64 processors and 500 to 512 segments: 13.4 ms on 313 wavefronts, 8.8 on 1024, 22 on 2048; 25,019
            // of 2 to 49 and 1 to 37 1.07 times as long on 512 as on 1024; 10,000 equal ones of 12 and 512 6.1 ms on 157, 6.0
            // on 512, 6.9 on 1024).  With at most 16 groups it goes on to all resident ones (3000 machines of 250 to 256
            // processors: 20.4 -> 13.7 ms, 15.4 on 1024).
            const int spread[2] = {total < kSIMDs ? total : kSIMDs, total};
            for (int k = 0; k < 2; ++k)
                G.parts.per_wave[k] = static_cast<int>(n > static_cast<int64_t>(spread[k]) * kWave ? kWave : (n + spread[k] - 1) / spread[k]);
            G.stream = st;
            if (launch_bi_group(G) != hipSuccess) return PRS_EDEVICE;
        } else if (general(c, P.order, k) != hipSuccess) {
            return PRS_EDEVICE;
        }
    }
    // bi-greedy configurations whose list of running groups did not fit go through the general kernel
    if (model == PRS_BI && general(lay.rerun, retry, kRetryClass) != hipSuccess) return PRS_EDEVICE;
    return PRS_OK;
}

// ---- best segmentation per algorithm: candidates q_req = 2^c, c < n_cand, for every problem ----------
template <typename T>
__global__ void search_expand(ConfigArrays in, int64_t n, int n_cand, int32_t *p, int32_t *q_req, int64_t *m, T *alpha, T *beta,
                              T *gamma)
{
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n * n_cand) return;
    const int64_t i = idx / n_cand;
    const int c = static_cast<int>(idx - i * n_cand);
    p[idx] = in.p[i];
    q_req[idx] = 1 << c;
    m[idx] = in.m[i];
    alpha[idx] = static_cast<const T *>(in.alpha)[i];
    beta[idx] = static_cast<const T *>(in.beta)[i];
    gamma[idx] = static_cast<const T *>(in.gamma)[i];
}

struct BestOut {
    void *T[4];
    int32_t *q[4];
    int32_t *cfg_status;
};

template <typename T>
__global__ void search_pick(int64_t n, int n_cand, const T *greedy, const T *pipeline, const T *binary, const T *revopt,
                            const int32_t *status, BestOut out)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const T *col[4] = {greedy, pipeline, binary, revopt};
    const int32_t st = status[i * n_cand];                         // the problem itself: candidate q_req = 1
    if (out.cfg_status) out.cfg_status[i] = st;
    for (int a = 0; a < 4; ++a) {
        T best = CostTraits<T>::bad();
        int32_t best_q = -1;
        if (st == PRS_CFG_OK) {
            for (int c = 0; c < n_cand; ++c) {
                if (status[i * n_cand + c] != PRS_CFG_OK) continue;
                const T v = col[a][i * n_cand + c];
                if (best_q < 0 || v < best) { best = v; best_q = 1 << c; }
            }
        }
        if (out.T[a]) static_cast<T *>(out.T[a])[i] = best;
        if (out.q[a]) out.q[a][i] = best_q;
    }
}

static int search_candidates(int32_t q_max)
{
    int c = 1;
    while ((INT64_C(1) << c) <= q_max) ++c;
    return c;                                                      // 1, 2, ..., 2^(c-1) <= q_max
}

struct SearchLayout {
    int n_cand;
    int64_t n_exp;
    size_t p, q_req, m, alpha, beta, gamma, greedy, pipeline, binary, revopt, status, sim, total;
};

static SearchLayout make_search_layout(int model, int64_t n, int32_t p_max, int32_t q_max)
{
    SearchLayout S;
    S.n_cand = search_candidates(q_max);
    S.n_exp = (n < 1 ? 1 : n) * S.n_cand;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += align256(bytes); return at; };
    const size_t e = static_cast<size_t>(S.n_exp);
    S.p = take(e * 4); S.q_req = take(e * 4); S.m = take(e * 8);
    S.alpha = take(e * 8); S.beta = take(e * 8); S.gamma = take(e * 8);
    S.greedy = take(e * 8); S.pipeline = take(e * 8); S.binary = take(e * 8); S.revopt = take(e * 8);
    S.status = take(e * 4);
    S.sim = off;
    S.total = off + make_layout(PRS_CALL_SIMULATE, model, S.n_exp, p_max, q_max).total;
    return S;
}

// ---- every segmentation of a short message (Section 8) --------------------------------------------
struct UnequalOut {
    void *T_best; uint32_t *cuts_best; int32_t *n_best;
    void *T_equi; uint32_t *cuts_equi; int32_t *equi_optimal; int32_t *cfg_status;
};

// Equal sizes except a last segment that may be smaller: returns that size, or 0 if the composition is not of this kind.
__device__ __forceinline__ int equal_but_last(uint32_t comp)
{
    const int s = comp_first(comp);
    comp >>= s;
    while (comp != 0) {
        const int z = comp_first(comp);
        comp >>= z;
        if (z != s && !(comp == 0 && z < s)) return 0;
    }
    return s;
}

constexpr int kPickThreads = 256;

// One block per problem: minima over its 2^(m-1) times, ties to the smallest cut pattern.
template <typename T>
__global__ __launch_bounds__(kPickThreads) void unequal_pick(ConfigArrays in, int32_t p_max, int32_t m_max, const T *times,
                                                             const int32_t *status, UnequalOut out)
{
    __shared__ T sBest[kPickThreads], sEqui[kPickThreads];
    __shared__ uint32_t sBestC[kPickThreads], sEquiC[kPickThreads];
    const int64_t i = blockIdx.x;
    const int tid = static_cast<int>(threadIdx.x);
    const int bits = m_max - 1;
    const int64_t base = i << bits;
    const int64_t m = in.m[i];
    const int32_t st = status[base];                               // pattern 0 is a segmentation of every valid problem
    if (st != PRS_CFG_OK) {
        if (tid == 0) {
            if (out.cfg_status) out.cfg_status[i] = st;
            if (out.T_best) static_cast<T *>(out.T_best)[i] = CostTraits<T>::bad();
            if (out.T_equi) static_cast<T *>(out.T_equi)[i] = CostTraits<T>::bad();
            if (out.cuts_best) out.cuts_best[i] = 0;
            if (out.cuts_equi) out.cuts_equi[i] = 0;
            if (out.n_best) out.n_best[i] = 0;
            if (out.equi_optimal) out.equi_optimal[i] = 0;
        }
        return;
    }
    const uint32_t n_comp = 1u << static_cast<int>(m - 1);
    const uint32_t closing = 1u << static_cast<int>(m - 1);
    const T kInf = CostTraits<T>::inf();
    T best = kInf, equi = kInf;
    uint32_t best_c = 0, equi_c = 0;
    for (uint32_t c = tid; c < n_comp; c += kPickThreads) {        // rising patterns: the first minimum is the smallest pattern
        const T v = times[base + c];
        if (v < best) { best = v; best_c = c; }
        const int s = equal_but_last(c | closing);
        // an equi-segmentation cut from a count k has size ceil(m/k): s is such a size iff ceil(m / ceil(m/s)) == s
        if (s > 0) {
            const int64_t k = (m + s - 1) / s;
            if ((m + k - 1) / k == s && v < equi) { equi = v; equi_c = c; }
        }
    }
    sBest[tid] = best; sBestC[tid] = best_c; sEqui[tid] = equi; sEquiC[tid] = equi_c;
    __syncthreads();
    for (int t = 0; t < kPickThreads; ++t) {                        // every thread folds the whole table: all end with the same minima
        const T b = sBest[t];
        if (b < best || (b == best && sBestC[t] < best_c)) { best = b; best_c = sBestC[t]; }
        const T e = sEqui[t];
        if (e < equi || (e == equi && sEquiC[t] < equi_c)) { equi = e; equi_c = sEquiC[t]; }
    }
    // second pass: how many segmentations reach the minimum, and whether one of them has equal sizes but the last
    int cnt = 0, wide = 0;
    for (uint32_t c = tid; c < n_comp; c += kPickThreads) {
        if (times[base + c] == best) {
            ++cnt;
            if (equal_but_last(c | closing) > 0) wide = 1;
        }
    }
    __shared__ int sCnt[kPickThreads], sWide[kPickThreads];
    sCnt[tid] = cnt; sWide[tid] = wide;
    __syncthreads();
    if (tid == 0) {
        int total = 0, any_wide = 0;
        for (int t = 0; t < kPickThreads; ++t) { total += sCnt[t]; any_wide |= sWide[t]; }
        if (out.cfg_status) out.cfg_status[i] = PRS_CFG_OK;
        if (out.T_best) static_cast<T *>(out.T_best)[i] = best;
        if (out.cuts_best) out.cuts_best[i] = best_c;
        if (out.n_best) out.n_best[i] = total;
        if (out.T_equi) static_cast<T *>(out.T_equi)[i] = equi;
        if (out.cuts_equi) out.cuts_equi[i] = equi_c;
        if (out.equi_optimal) out.equi_optimal[i] = (equi == best ? 1 : 0) | (any_wide ? 2 : 0);
    }
}

struct UnequalLayout {
    int64_t n_exp;
    size_t times, status, sim, total;
};

static UnequalLayout make_unequal_layout(int64_t n, int32_t p_max, int32_t m_max)
{
    UnequalLayout U;
    U.n_exp = (n < 1 ? 1 : n) << (m_max - 1);
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += align256(bytes); return at; };
    U.times = take(static_cast<size_t>(U.n_exp) * 8);
    U.status = take(static_cast<size_t>(U.n_exp) * 4);
    U.sim = off;
    U.total = off + make_layout(PRS_CALL_SIMULATE, PRS_UNI, U.n_exp, p_max, m_max, nullptr, true).total;
    return U;
}

constexpr int kUnequalMaxM = 24;

}  // namespace prs

using namespace prs;

extern "C" {

int prs_abi_version(void) { return 2; }

size_t prs_workspace_bytes(int call, int model, int cost, int64_t n, int32_t p_max, int32_t q_max)
{
    (void)cost;
    if (n < 0 || p_max < 2 || q_max < 1) return 0;
    if (call == PRS_CALL_REPLAY) return replay_workspace_bytes(p_max, q_max);
    if (call == PRS_CALL_OFFSETS) return kHeaderBytes;
    if (call == PRS_CALL_SEARCH) return make_search_layout(model, n, p_max, q_max).total;
    if (call == PRS_CALL_UNEQUAL) {
        if (q_max > kUnequalMaxM || (n << (q_max - 1)) >= (INT64_C(1) << 31)) return 0;
        return make_unequal_layout(n, p_max, q_max).total;
    }
    if (call != PRS_CALL_SIMULATE && call != PRS_CALL_SCHEDULE) return 0;
    return make_layout(call, model, n, p_max, q_max).total;
}

int simulate_completion_batch(const prs_configs *cfg, int64_t n, int model, int cost, int32_t p_max, int32_t q_max,
                              const prs_times *out, void *workspace, size_t workspace_bytes, void *stream,
                              const prs_tuning *tuning)
{
    if (bad_common(cfg, n, model, cost, p_max, q_max) || !out) return PRS_EINVAL;
    TimesOut t{out->greedy, out->binomial, out->pipeline, out->binary, out->revopt,
               out->butterfly, out->lower_bound, out->q_eff, out->cfg_status};
    SchedOut s{};
    return run_greedy(PRS_CALL_SIMULATE, cfg, n, model, cost, p_max, q_max, t, s, workspace, workspace_bytes, stream, tuning);
}

int optimal_segmentation_batch(const prs_configs *cfg, int64_t n, int model, int cost, int32_t p_max, int32_t q_max,
                               const prs_best *out, void *workspace, size_t workspace_bytes, void *stream,
                               const prs_tuning *tuning)
{
    if (!cfg || !out || n < 0 || n >= (INT64_C(1) << 26) || (model != PRS_UNI && model != PRS_BI) ||
        (cost != PRS_COST_I64 && cost != PRS_COST_F64) || p_max < 2 || p_max > (1 << 20) || q_max < 1 || q_max > (1 << 20))
        return PRS_EINVAL;
    if (n > 0 && (!cfg->p || !cfg->m || !cfg->alpha || !cfg->beta || !cfg->gamma)) return PRS_EINVAL;
    if (n == 0) return PRS_OK;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return PRS_EINVAL;
    const SearchLayout S = make_search_layout(model, n, p_max, q_max);
    if (workspace_bytes < S.total) return PRS_ENOSPC;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const ConfigArrays in{cfg->p, nullptr, cfg->m, cfg->alpha, cfg->beta, cfg->gamma};
    int32_t *ep = reinterpret_cast<int32_t *>(ws + S.p), *eq = reinterpret_cast<int32_t *>(ws + S.q_req);
    int64_t *em = reinterpret_cast<int64_t *>(ws + S.m);
    const int64_t n_exp = n * S.n_cand;
    const unsigned blocks = static_cast<unsigned>((n_exp + 255) / 256);
    if (cost == PRS_COST_I64)
        hipLaunchKernelGGL((search_expand<int64_t>), dim3(blocks), dim3(256), 0, st, in, n, S.n_cand, ep, eq, em,
                           reinterpret_cast<int64_t *>(ws + S.alpha), reinterpret_cast<int64_t *>(ws + S.beta),
                           reinterpret_cast<int64_t *>(ws + S.gamma));
    else
        hipLaunchKernelGGL((search_expand<double>), dim3(blocks), dim3(256), 0, st, in, n, S.n_cand, ep, eq, em,
                           reinterpret_cast<double *>(ws + S.alpha), reinterpret_cast<double *>(ws + S.beta),
                           reinterpret_cast<double *>(ws + S.gamma));
    if (hipGetLastError() != hipSuccess) return PRS_EDEVICE;
    const prs_configs exp_cfg{ep, eq, em, ws + S.alpha, ws + S.beta, ws + S.gamma};
    TimesOut t{ws + S.greedy, nullptr, ws + S.pipeline, ws + S.binary, ws + S.revopt, nullptr, nullptr, nullptr,
               reinterpret_cast<int32_t *>(ws + S.status)};
    SchedOut s{};
    const int rc = run_greedy(PRS_CALL_SIMULATE, &exp_cfg, n_exp, model, cost, p_max, q_max, t, s, ws + S.sim,
                              workspace_bytes - S.sim, stream, tuning);
    if (rc != PRS_OK) return rc;
    BestOut b{{out->T_greedy, out->T_pipeline, out->T_binary, out->T_revopt},
              {out->q_greedy, out->q_pipeline, out->q_binary, out->q_revopt}, out->cfg_status};
    const unsigned pblocks = static_cast<unsigned>((n + 255) / 256);
    if (cost == PRS_COST_I64)
        hipLaunchKernelGGL((search_pick<int64_t>), dim3(pblocks), dim3(256), 0, st, n, S.n_cand,
                           reinterpret_cast<const int64_t *>(ws + S.greedy), reinterpret_cast<const int64_t *>(ws + S.pipeline),
                           reinterpret_cast<const int64_t *>(ws + S.binary), reinterpret_cast<const int64_t *>(ws + S.revopt),
                           reinterpret_cast<const int32_t *>(ws + S.status), b);
    else
        hipLaunchKernelGGL((search_pick<double>), dim3(pblocks), dim3(256), 0, st, n, S.n_cand,
                           reinterpret_cast<const double *>(ws + S.greedy), reinterpret_cast<const double *>(ws + S.pipeline),
                           reinterpret_cast<const double *>(ws + S.binary), reinterpret_cast<const double *>(ws + S.revopt),
                           reinterpret_cast<const int32_t *>(ws + S.status), b);
    return hipGetLastError() == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int unequal_segmentation_batch(const prs_configs *cfg, int64_t n, int cost, int32_t p_max, int32_t m_max,
                               const prs_unequal *out, void *workspace, size_t workspace_bytes, void *stream,
                               const prs_tuning *tuning)
{
    if (!cfg || !out || n < 0 || (cost != PRS_COST_I64 && cost != PRS_COST_F64) || p_max < 2 || p_max > (1 << 20) ||
        m_max < 1 || m_max > kUnequalMaxM || (n << (m_max - 1)) >= (INT64_C(1) << 31))
        return PRS_EINVAL;
    if (n > 0 && (!cfg->p || !cfg->m || !cfg->alpha || !cfg->beta || !cfg->gamma)) return PRS_EINVAL;
    if (n == 0) return PRS_OK;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return PRS_EINVAL;
    const UnequalLayout U = make_unequal_layout(n, p_max, m_max);
    if (workspace_bytes < U.total) return PRS_ENOSPC;
    char *ws = static_cast<char *>(workspace);
    void *all = out->T_all ? out->T_all : static_cast<void *>(ws + U.times);
    int32_t *status = reinterpret_cast<int32_t *>(ws + U.status);
    const prs_configs problems{cfg->p, nullptr, cfg->m, cfg->alpha, cfg->beta, cfg->gamma};
    TimesOut t{all, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, status};
    SchedOut s{};
    const int rc = run_greedy(PRS_CALL_SIMULATE, &problems, U.n_exp, PRS_UNI, cost, p_max, m_max, t, s, ws + U.sim,
                              workspace_bytes - U.sim, stream, tuning, m_max);
    if (rc != PRS_OK) return rc;
    const ConfigArrays in{cfg->p, nullptr, cfg->m, cfg->alpha, cfg->beta, cfg->gamma};
    const UnequalOut u{out->T_best, out->cuts_best, out->n_best, out->T_equi, out->cuts_equi, out->equi_optimal, out->cfg_status};
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (cost == PRS_COST_I64)
        hipLaunchKernelGGL((unequal_pick<int64_t>), dim3(static_cast<unsigned>(n)), dim3(kPickThreads), 0, st, in, p_max, m_max,
                           static_cast<const int64_t *>(all), status, u);
    else
        hipLaunchKernelGGL((unequal_pick<double>), dim3(static_cast<unsigned>(n)), dim3(kPickThreads), 0, st, in, p_max, m_max,
                           static_cast<const double *>(all), status, u);
    return hipGetLastError() == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int butterfly_threshold_batch(const int32_t *p, int64_t n, double alpha, int32_t q_max, int32_t m_log2_first,
                              int32_t m_log2_last, double ratio_lo, double ratio_hi, int32_t steps, double *ratio_below,
                              double *ratio_above, int32_t *cfg_status, void *stream)
{
    if (n < 0 || n >= (INT64_C(1) << 31) || (n > 0 && !p) || q_max < 1 || q_max > (1 << 20) || m_log2_first < 0 ||
        m_log2_last < m_log2_first || m_log2_last > 40 || steps < 0 || steps > 64)
        return PRS_EINVAL;
    if (!(alpha >= 0.0) || !(alpha < 1e300) || !(ratio_lo > 0.0) || !(ratio_hi > ratio_lo) || !(ratio_hi < 1e100)) return PRS_EINVAL;
    if (n == 0) return PRS_OK;
    ThresholdLaunch L{p, n, alpha, q_max, m_log2_first, m_log2_last, ratio_lo, ratio_hi, steps, ratio_below, ratio_above,
                      cfg_status, static_cast<hipStream_t>(stream)};
    return launch_threshold(L) == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int prs_measure_alu_ceiling(int64_t steps_per_lane, int32_t blocks, double *sink, void *stream)
{
    if (steps_per_lane < 0 || blocks < 1 || blocks > (1 << 20) || !sink) return PRS_EINVAL;
    return launch_alu_ceiling(steps_per_lane, blocks, sink, static_cast<hipStream_t>(stream)) == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int prs_pair_offsets(const prs_configs *cfg, int64_t n, int cost, int32_t p_max, int32_t q_max, int64_t *pair_offset,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    (void)workspace; (void)workspace_bytes;
    if (bad_common(cfg, n, PRS_UNI, cost, p_max, q_max) || !pair_offset) return PRS_EINVAL;
    OffsetsLaunch L{ConfigArrays{cfg->p, cfg->q_req, cfg->m, cfg->alpha, cfg->beta, cfg->gamma}, n, p_max, q_max, cost,
                    pair_offset, static_cast<hipStream_t>(stream)};
    return launch_offsets(L) == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int greedy_schedule_batch(const prs_configs *cfg, int64_t n, int model, int cost, int32_t p_max, int32_t q_max,
                          const int64_t *pair_offset, int64_t pair_capacity, int32_t *src, int32_t *dst, int32_t *seg,
                          void *t_start, void *T_greedy, int32_t *cfg_status, void *workspace, size_t workspace_bytes,
                          void *stream, const prs_tuning *tuning)
{
    if (bad_common(cfg, n, model, cost, p_max, q_max) || pair_capacity < 0 || (n > 0 && !pair_offset)) return PRS_EINVAL;
    TimesOut t{};
    SchedOut s{pair_offset, pair_capacity, src, dst, seg, t_start, T_greedy, cfg_status};
    return run_greedy(PRS_CALL_SCHEDULE, cfg, n, model, cost, p_max, q_max, t, s, workspace, workspace_bytes, stream, tuning);
}

// argument checks shared by the two replay entry points
static int replay_bad_arguments(int32_t p, int32_t q, const int64_t *seg_elem_offset, const int32_t *src, const int32_t *dst,
                                const int32_t *seg, int64_t n_pairs, const void *in, int64_t stride_elems, int64_t n_elems,
                                int dtype, const void *out)
{
    if (p < 2 || p > 4096 || q < 1 || q > 65536 || !seg_elem_offset || !src || !dst || !seg || !in || !out) return PRS_EINVAL;
    if (n_pairs != static_cast<int64_t>(p - 1) * q || n_pairs >= (INT64_C(1) << 31)) return PRS_EINVAL;
    const int elem = dtype & 0xFF, op = dtype & ~0xFF;
    if ((elem != PRS_I32 && elem != PRS_F32 && elem != PRS_F64 && elem != PRS_I64) || (op != PRS_OP_SUM && op != PRS_OP_MAX))
        return PRS_EINVAL;
    if (n_elems < 0 || stride_elems < n_elems) return PRS_EINVAL;
    if (seg_elem_offset[0] != 0 || seg_elem_offset[q] != n_elems) return PRS_EINVAL;
    for (int k = 0; k < q; ++k)
        if (seg_elem_offset[k + 1] < seg_elem_offset[k]) return PRS_EINVAL;
    return PRS_OK;
}

int replay_reduction_static(int32_t p, int32_t q, const int64_t *seg_elem_offset, const int32_t *src, const int32_t *dst,
                            const int32_t *seg, int64_t n_pairs, const void *in, int64_t stride_elems, int64_t n_elems,
                            int dtype, void *out, int32_t *status, void *stream)
{
    const int bad = replay_bad_arguments(p, q, seg_elem_offset, src, dst, seg, n_pairs, in, stride_elems, n_elems, dtype, out);
    if (bad != PRS_OK) return bad;
    if (replay_scratch_bytes(p, q) > kReplayStaticBytes) return PRS_ENOSPC;       // too many processors x segments for the fixed array
    void *ws = nullptr;
    if (replay_static_scratch(&ws) != hipSuccess) return PRS_EDEVICE;
    ReplayLaunch L{p, q, seg_elem_offset, src, dst, seg, n_pairs, in, stride_elems, n_elems, dtype & 0xFF, dtype & ~0xFF, out, status,
                   static_cast<char *>(ws), static_cast<hipStream_t>(stream)};
    return launch_replay(L) == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

int replay_reduction(int32_t p, int32_t q, const int64_t *seg_elem_offset, const int32_t *src, const int32_t *dst,
                     const int32_t *seg, int64_t n_pairs, const void *in, int64_t stride_elems, int64_t n_elems, int dtype,
                     void *out, int32_t *status, void *workspace, size_t workspace_bytes, void *stream)
{
    if (p < 2 || p > 4096 || q < 1 || q > 65536 || !seg_elem_offset || !src || !dst || !seg || !in || !out) return PRS_EINVAL;
    if (n_pairs != static_cast<int64_t>(p - 1) * q || n_pairs >= (INT64_C(1) << 31)) return PRS_EINVAL;
    const int elem = dtype & 0xFF, op = dtype & ~0xFF;
    if ((elem != PRS_I32 && elem != PRS_F32 && elem != PRS_F64 && elem != PRS_I64) || (op != PRS_OP_SUM && op != PRS_OP_MAX))
        return PRS_EINVAL;
    if (n_elems < 0 || stride_elems < n_elems) return PRS_EINVAL;
    if (seg_elem_offset[0] != 0 || seg_elem_offset[q] != n_elems) return PRS_EINVAL;
    for (int k = 0; k < q; ++k)
        if (seg_elem_offset[k + 1] < seg_elem_offset[k]) return PRS_EINVAL;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return PRS_EINVAL;
    if (workspace_bytes < replay_workspace_bytes(p, q)) return PRS_ENOSPC;
    ReplayLaunch L{p, q, seg_elem_offset, src, dst, seg, n_pairs, in, stride_elems, n_elems, elem, op, out, status,
                   static_cast<char *>(workspace), static_cast<hipStream_t>(stream)};
    return launch_replay(L) == hipSuccess ? PRS_OK : PRS_EDEVICE;
}

}  // extern "C"
