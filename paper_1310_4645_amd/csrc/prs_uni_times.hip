// Uni-greedy completion times (Lowery & Langou, Algorithm 1, Section 5) on gfx950: segments pipelined
// through the lanes of a wavefront, equal ready times handled as one run.
//
// Algorithm 1 handles segment k+1 with the final states of segment k as its initial states, but it only
// ever looks at the smallest of them.  The states of segment k leave in non-decreasing order (the start
// time t of its pairs never decreases), so segment k+1 can begin as soon as segment k has produced its
// first values and then follows right behind it.  A configuration is given a group of G lanes (1 to 64,
// chosen from its number of pairs); lane l of the group runs segments l, l+G, l+2G, ... and reads the
// stream written by the lane before it (lane 0 the stream of the last lane, one round earlier).
//
// Many processors share a ready time, and which of them is which does not enter any time.  Streams
// therefore hold runs (value, how many processors), and a step of a segment takes a whole run: of n
// processors ready at v, with r = 0 or 1 left over from an earlier value, (r + n) / 2 pairs start at v,
// send until v + tcomm (a run of the output stream) and combine until (v + tcomm) + tcomp (a run of B, the
// receivers that come back), and (r + n) mod 2 are left over.  The runs a segment has left are the unread
// tail of its input stream A merged with the unread tail of B; both are sorted, so a step compares two
// heads.  On the sweep up to 1024 processors a step stands for 1.9 pairs on average (3 above 512), with
// tens of thousands of processors for 5 to 130.  Taking a run in two pieces gives the same pairs, so runs
// of equal value need not be joined; the newest run of a stream is joined with the next one if their values
// are equal (different start times can round to the same sum), which saves a fifth of the steps.
//
// B is not stored: B[i] = stream[i] + tcomp with the same rounding as (t + tcomm) + tcomp.  The root's
// final state (the largest value of the segment) closes the stream of a segment.  A stream is published
// up to its newest run, which is still open; the value of the open run (0 before the first) is a lower
// bound of everything that follows, so a reader that has nothing left may take a value of B below it.
//
// Every stream lives in a ring in LDS and nothing of it in global memory: a lane whose ring is full
// waits for its reader and for its own B.  (With the streams backed by global memory the kernel was bound by
// the scattered 8-byte stores, about 9 cycles of a CU's store path each.)  The rings of a group can all be
// full at once only through the last lane, whose reader, the first lane, is a whole round behind: its ring
// is the deep one.  If it does fill up -- or B outgrows a ring -- no lane of the group moves any more; the
// configuration then starts again with its rings in the wavefront's workspace slot, p + 7 runs each (none where p + 7 runs fit
// every ring in LDS), in which a lane never waits: of its stream at most p runs are unread -- a segment cannot have sent more processors than
// the lane that reads its stream has taken from the stream before it, and all p of them with one lane, which
// reads its own stream, at the end of a segment without equal ready times -- and a lane goes on as long as 7 places
// are left, for the runs of a chunk of steps, the root's and the open one.  (p + 4 places were too few for one lane.)
//
// Measured (pair by pair with streams in global memory -> runs in LDS rings -> 27 KB of rings, five wavefronts per CU instead
// of four, and tickets drawn several at a time): the 100,000-configuration sweep 11.9 -> 4.1 -> 3.55 ms, 64 machines of
// 1024 to 65536 processors 587 -> 7.4 -> 7.0 ms, 986 x 512 segmentations of a short message 10.4 -> 1.94 -> 1.43 ms.  A step is
// about 65 instructions, a chain of an LDS read, two compares and two additions, and takes 240 ns on a SIMD of its own:
// that latency is what bounds it, with one or two wavefronts per SIMD.
#include "prs_device.h"
#include "prs_launch.h"

namespace prs {

constexpr int kMaxChunk = 4;                     // steps between two looks for room in a ring, at most
constexpr int kSpan = 64;                        // steps between two looks for groups that do not move
constexpr int kRunBytes = 12;                    // a run in a ring: value and count
constexpr int32_t kRetired = 1 << 30;            // read place of a lane without a segment: its producer need not wait for it

template <typename T> struct __attribute__((packed, aligned(4))) Run { T v; int32_t n; };

// Machines of up to 1024 processors: counts fit 16 bits, and a wavefront keeps its runs in 27 KB, values first: five
// wavefronts per CU (LDS is given out in units of 1280 bytes).  B has at most 23 runs on all but a dozen of the 100,000-configuration sweep, and 30 - 3 - 4 of a ring of
// 30 can wait (the root's run, the open place, the runs of four steps).  Compositions, whose segments differ in size,
// keep more runs waiting: 40 KB, four wavefronts per CU.
template <bool kComp> struct SmallRings;
template <> struct SmallRings<false> { static constexpr int kRuns = 2730, kRing = 30; };
template <> struct SmallRings<true> { static constexpr int kRuns = 4096, kRing = 36; };
static RingShape large_rings(int32_t p_max)
{
    return p_max <= kUniMidProcs ? RingShape{6826, 96} : RingShape{13653, 192};       // B: 40 runs with 15,000 processors, 131 with 45,000
}
size_t uni_times_lds_bytes(int32_t p_max, bool compositions)
{
    if (p_max <= kUniSmallProcs) return static_cast<size_t>(compositions ? SmallRings<true>::kRuns : SmallRings<false>::kRuns) * 10;
    return static_cast<size_t>(large_rings(p_max).runs) * kRunBytes;
}
// runs of a ring in the workspace: none for machines that never fill one in LDS
int32_t uni_times_slot_runs(int32_t p_max)
{
    static_assert(SmallRings<false>::kRing <= SmallRings<true>::kRing, "the smallest ring in LDS");
    const int32_t runs = p_max + 3 + kMaxChunk;
    return runs <= SmallRings<false>::kRing ? 0 : (runs + 1) / 2 * 2;
}
// Packed like the large rings for compositions as well, many of which start again (the two loads of a run whose count lies apart
// cost 78 x 2048 of them 2.01 ms against 1.85); apart where few do and there are the most wavefronts.
size_t uni_times_slot_bytes(int32_t runs, bool packed) { return static_cast<size_t>(kWave) * static_cast<size_t>(runs) * (packed ? kRunBytes : 10); }

// Runs in LDS by the byte address of their place.  kSmall: the value there, the count among the 16-bit ones behind all
// values; otherwise both packed into 12 bytes.
// kSmallRuns: how many runs a wavefront keeps, 0 if they are packed
template <typename T, int kSmallRuns> __device__ __forceinline__ void lds_load(int32_t at, T &v, int32_t &n)
{
    if (kSmallRuns > 0) { v = *lds_at<T>(at); n = *lds_at<uint16_t>((at >> 2) + kSmallRuns * 8); }
    else { const auto *e = lds_at<Run<T>>(at); v = e->v; n = e->n; }
}
template <typename T, int kSmallRuns> __device__ __forceinline__ void lds_value(int32_t at, T &v)
{
    if (kSmallRuns > 0) v = *lds_at<T>(at);
    else v = lds_at<Run<T>>(at)->v;
}
template <typename T, int kSmallRuns> __device__ __forceinline__ void lds_count(int32_t at, int32_t &n)
{
    if (kSmallRuns > 0) n = *lds_at<uint16_t>((at >> 2) + kSmallRuns * 8);
    else n = lds_at<Run<T>>(at)->n;
}
template <typename T, int kSmallRuns> __device__ __forceinline__ void lds_store(int32_t at, T v, int32_t n)
{
    if (kSmallRuns > 0) { *lds_at<T>(at) = v; *lds_at<uint16_t>((at >> 2) + kSmallRuns * 8) = static_cast<uint16_t>(n); }
    else { auto *e = lds_at<Run<T>>(at); e->v = v; e->n = n; }
}

// A ring of runs at byte addresses base, base + stride, ..., end (exclusive) of LDS or of the workspace slot.
struct Ring { int32_t base, stride, end; };

// Rings of a wavefront in LDS: the last lane of every group has a deep ring, the others s.runs_per_lane runs.
// Both kinds are laid out run by run, the lanes side by side, so that lanes at different places of their rings mostly
// stay on different banks.
template <int G, bool kSmall> __device__ __forceinline__ Ring lds_ring(int l, const RingShape &s)
{
    constexpr int kBytes = kSmall ? 8 : kRunBytes, kGroups = kWave / G, kCols = G == 1 ? 0 : (G >= 8 ? kWave : kWave - kGroups);
    const int g = l / G, i = l & (G - 1), shallow = kCols * s.runs_per_lane;
    int runs = s.runs_per_lane;
    Ring r;
    if (i == G - 1) {
        r.base = (shallow + g) * kBytes; r.stride = kGroups * kBytes; runs = (s.runs - shallow) / kGroups;
    } else {
        r.base = (G >= 8 ? l : g * (G - 1) + i) * kBytes; r.stride = kCols * kBytes;
    }
    r.end = r.base + runs * r.stride;
    return r;
}
template <bool kPacked> __device__ __forceinline__ Ring slot_ring(int l, int32_t slot_runs)
{
    constexpr int kBytes = kPacked ? kRunBytes : 8;
    Ring r;
    r.base = l * slot_runs * kBytes; r.stride = kBytes; r.end = r.base + slot_runs * kBytes;
    return r;
}
// runs in the workspace slot, packed or with their 16-bit counts from `counts` on
template <typename T, bool kPacked> __device__ __forceinline__ void slot_load(const char *slot, int32_t counts, int32_t at, T &v, int32_t &n)
{
    if (!kPacked) { v = *reinterpret_cast<const T *>(slot + at); n = *reinterpret_cast<const uint16_t *>(slot + counts + (at >> 2)); }
    else { const auto *e = reinterpret_cast<const Run<T> *>(slot + at); v = e->v; n = e->n; }
}
template <typename T, bool kPacked> __device__ __forceinline__ void slot_store(char *slot, int32_t counts, int32_t at, T v, int32_t n)
{
    if (!kPacked) { *reinterpret_cast<T *>(slot + at) = v; *reinterpret_cast<uint16_t *>(slot + counts + (at >> 2)) = static_cast<uint16_t>(n); }
    else { auto *e = reinterpret_cast<Run<T> *>(slot + at); e->v = v; e->n = n; }
}
__device__ __forceinline__ int32_t ring_next(const Ring &r, int32_t at)
{
    const int32_t n = at + r.stride;
    return n == r.end ? r.base : n;
}

// kComp: the segments of a configuration have the sizes its composition gives (Section 8) instead of one size
// and a smaller last one; every lane keeps the part of the composition that starts at its segment.
template <typename T, int G, bool kComp, bool kSmall>
__device__ __forceinline__ void uni_times_body(const RingShape &shape, const ConfigArrays &cfg, int32_t p_max, int32_t q_max,
                                               int model, const TimesOut &times, PlanHeader *plan, const int32_t *order, int cls,
                                               int part, char *slot, int32_t slot_runs, bool help = false)
{
    constexpr int kGroups = kWave / G, kSmallRuns = kSmall ? SmallRings<kComp>::kRuns : 0;
    constexpr bool kPacked = kComp || !kSmall;      // runs in the workspace slot
    // a new configuration is fetched (a path every lane waits for) when this many groups have nothing to do
    constexpr int kFetchGroups = kGroups >= 8 ? kGroups / 8 : 1;
    // steps between two looks for room in the ring and for the end of a segment (small groups have short segments)
    constexpr int kChunk = G >= 8 ? kMaxChunk : 2;
    const int lane = lane_id(), gl = lane & (G - 1), gbase = lane & ~(G - 1);
    const int prod = gbase | ((gl + G - 1) & (G - 1));
    const uint64_t gmask = (G == 64 ? ~UINT64_C(0) : ((UINT64_C(1) << G) - 1)) << gbase;
    // part of the class this pass works on: all of it, its giant configurations only, or the rest after those
    const int set = cls >= kLargeClass ? 1 : 0;
    const int32_t counts = kWave * 8 * slot_runs;                     // unless kPacked: where they begin in the slot
    int32_t count = plan->class_count[cls], begin = plan->class_begin[cls];
    unsigned long long *tickets = &plan->ticket[cls];
    if (part == kGiantPart) { count = plan->giant_count[set]; tickets = &plan->ticket_giant[set]; }
    else if (part == kRestPart) { begin += plan->giant_count[set]; count -= plan->giant_count[set]; }
    if (count == 0) return;
    // Tickets are drawn several at a time, a sixteenth of a wavefront's share at most (a counter that every wavefront adds to
    // serves one of them every few nanoseconds); those in hand are hand .. hand_end - 1, and may lie past the end.
    int batch = count / (static_cast<int>(gridDim.x) * 16);
    if (batch > 4 * kGroups) batch = 4 * kGroups;
    if (help) batch = 0;                                              // every ticket drawn is run
    int64_t hand = 0, hand_end = 0;

    // ---- per-group state (the same in all lanes of a group)
    bool have = false, exhausted = false, in_slot = false;
    int64_t ci = 0;
    int p = 2, q = 1;
    T c_full = 0, g_full = 0, c_last = 0, g_last = 0;
    T alpha = 0, beta = 0, gamma = 0;   // kComp only
    uint32_t comp = 0, rest = 0;        // kComp only: the composition; the part of it from my segment on (per lane)
    // ---- per-lane state
    Ring own = lds_ring<G, kSmall>(lane, shape), in = lds_ring<G, kSmall>(prod, shape);    // my output stream, my input stream
    bool active = false;            // this lane has a segment to run
    int k = 0;                      // which one
    int left = 0;                   // pairs it still has to form
    int aleft = 0;                  // processors of my input stream not taken yet
    int32_t aat = 0, bat = 0;       // places of the heads of A (in my producer's ring) and B (in mine)
    int32_t wat = 0, wlast = 0;     // place of the next run to write; of the newest one (wat if the segment has none): published before it
    int odd = 0;                    // processor left over from an earlier value
    T lastS = 0, cc = 0, gg = 0;    // value of the newest run (-1: none in this segment), costs of my segment
    int lastN = 0;                  // its count

    auto put = [&](auto to_slot, int32_t at, T v, int n) {
        if (decltype(to_slot)::value) {
            slot_store<T, kPacked>(slot, counts, at, v, n);
        } else {
            lds_store<T, kSmallRuns>(at, v, n);
        }
    };
    auto segment_costs = [&]() {
        cc = k == q - 1 ? c_last : c_full; gg = k == q - 1 ? g_last : g_full;
        if (kComp) {
            const T sz = static_cast<T>(rest ? comp_first(rest) : 1);
            const T bs = beta * sz;                                          // each product and sum rounded on its own
            cc = alpha + bs; gg = gamma * sz;
        }
    };
    // first segment of every lane; the input stream of segment 0 is p processors at time 0
    auto start_configuration = [&](auto to_slot) {
        k = gl; active = k < q;
        left = active ? p - 1 : 0; aleft = p; odd = 0; lastS = T(-1); lastN = 0;
        aat = in.base;
        wat = own.base;
        if (gl == G - 1) { put(to_slot, wat, T(0), p); wat = ring_next(own, wat); }
        put(to_slot, wat, T(0), 0);
        bat = wlast = wat;
        if (kComp) rest = comp_drop(comp, gl);
        segment_costs();
    };

    for (;;) {
        // ---------------------------------------------------------------- fetch configurations
        if (help && __hip_atomic_load(&plan->large_left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) exhausted = exhausted || !have;
        const uint64_t need = ballot64(gl == 0 && !have && !exhausted);
        if (need != 0) {
            // the groups without a configuration take the tickets in hand first, then those just drawn
            const int wanted = __builtin_popcountll(need), in_hand = static_cast<int>(hand_end - hand);
            const int more = wanted - in_hand, grab = more > batch ? more : batch;
            int64_t drawn = 0;
            if (more > 0) {
                const unsigned long long got = atomicAdd(tickets, lane == 0 ? static_cast<unsigned long long>(grab) : 0ULL);
                const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(got)),
                               hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(got >> 32));
                drawn = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
            }
            if (!have && !exhausted) {
                const int rank = __builtin_popcountll(need & ((UINT64_C(1) << gbase) - 1));
                const int64_t ticket = rank < in_hand ? hand + rank : drawn + (rank - in_hand);
                if (ticket >= count) {
                    exhausted = true;
                } else {
                    ci = order[begin + ticket];
                    const Config<T> c = decode_config<T>(cfg, ci, p_max, q_max);
                    if (gl == 0) {
                        if (!kComp) write_closed_forms<T>(times, ci, c, model);
                        if (times.cfg_status) times.cfg_status[ci] = c.status;
                        if (c.status != PRS_CFG_OK && times.greedy) static_cast<T *>(times.greedy)[ci] = CostTraits<T>::bad();
                    }
                    if (c.status == PRS_CFG_OK) {
                        have = true; in_slot = false;
                        p = c.p; q = c.q;
                        c_full = c.c_full; g_full = c.g_full; c_last = c.c_last; g_last = c.g_last;
                        if (kComp) { alpha = c.alpha; beta = c.beta; gamma = c.gamma; comp = c.comp; }
                        own = lds_ring<G, kSmall>(lane, shape); in = lds_ring<G, kSmall>(prod, shape);
                        start_configuration(BoolConst<false>());
                    }
                }
            }
            hand = more > 0 ? drawn + more : hand + wanted;
            if (more > 0) hand_end = drawn + grab;
        }
        if (ballot64(have) == 0 && ballot64(!exhausted) == 0) break;

        // ---------------------------------------------------------------- steps
        bool moved = false;
        auto steps = [&](auto with_slots) {
            constexpr bool kSlots = decltype(with_slots)::value;      // some lanes have their rings in the workspace slot
            auto store = [&](int32_t at, T v, int n) {
                if (kSlots && in_slot) put(BoolConst<true>(), at, v, n); else put(BoolConst<false>(), at, v, n);
            };
            __builtin_amdgcn_s_waitcnt(0);                            // nothing in the loop waits for what was asked for before it
            for (int it = 0; it < kSpan; it += kChunk) {
                // ---- is there room in my ring for the runs of a chunk of steps, the root's and the open place?
                const int32_t reader = from_next<G>(active ? aat : kRetired, gl);
                int32_t held = wat - reader, heldB = wat - bat;       // bytes of the ring not read yet
                if (held < 0) held += own.end - own.base;
                if (heldB < 0) heldB += own.end - own.base;
                if (reader == kRetired) held = 0;
                const int32_t most = own.end - own.base - (3 + kChunk) * own.stride;
                const bool room = held <= most && heldB <= most;
#pragma unroll
                for (int c = 0; c < kChunk; ++c) {
                    // ---- the heads of A and B
                    const int32_t upto = from_previous<G>(wlast, gl); // my producer has published its stream up to here
                    T va, vb;
                    int na, nb;
                    if (kSlots && in_slot) {
                        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");      // stores of earlier steps have landed
                        slot_load<T, kPacked>(slot, counts, aat, va, na);
                        slot_load<T, kPacked>(slot, counts, bat, vb, nb);
                    } else {
                        lds_value<T, kSmallRuns>(aat, va);
                        lds_value<T, kSmallRuns>(bat, vb);
                        asm volatile("" ::: "memory");                // the values first: the counts come while they are compared (sweep 3.45 -> 3.41 ms)
                        lds_count<T, kSmallRuns>(aat, na);
                        lds_count<T, kSmallRuns>(bat, nb);
                    }
                    asm volatile("" : "+v"(va), "+v"(vb) : : "memory");              // the loads stay outside the branches below
                    const bool avail = aat != upto;                   // else va is the value of the open run: a bound of what follows
                    const T a = or_absent<T>(aleft > 0, va), b = or_absent<T>(bat != wat, wrap_add<T>(vb, gg));
                    const bool le = a <= b, ge = b <= a, go = room & (left > 0);
                    const bool takeA = go & avail & le, takeB = go & ge & (avail | !le);
                    asm volatile("" : "+v"(na), "+v"(nb));
                    const int an = takeA ? na : 0, x = odd + an + (takeB ? nb : 0), pairs = x >> 1;
                    odd = x & 1;
                    aleft -= an;
                    aat = takeA ? ring_next(in, aat) : aat;
                    bat = takeB ? ring_next(own, bat) : bat;
                    moved = moved | takeA | takeB;
                    // ---- the pairs that start now: a run of my stream, or more of its newest run (unless B has taken that)
                    const T tc = wrap_add<T>(takeA ? a : b, cc);
                    const bool some = pairs > 0, join = some & (tc == lastS) & (bat != wat), fresh = some & !join;
                    const int n = pairs + (join ? lastN : 0);
                    wlast = fresh ? wat : wlast;
                    wat = fresh ? ring_next(own, wat) : wat;
                    left -= pairs;
                    if (some) { store(wlast, tc, n); lastS = tc; lastN = n; }
                }
                // ---- end of a segment
                const bool seg_end = active && left == 0;
                if (ballot64(seg_end) != 0) {
                    PRS_KEEP_BRANCH();
                    if (seg_end) {
                        const T tr = wrap_add<T>(lastS, gg);                // the last receiver is the root
                        if (tr == lastS) { store(wlast, tr, lastN + 1); }
                        else { store(wat, tr, 1); wat = ring_next(own, wat); }
                        store(wat, T(0), 0);
                        bat = wlast = wat;
                        if (k == q - 1 && times.greedy) static_cast<T *>(times.greedy)[ci] = tr;
                        if (!kSmall && k == q - 1 && set == 1) atomicAdd(&plan->large_left, -1);
                        k += G;
                        active = k < q;
                        lastS = T(-1); odd = 0; left = active ? p - 1 : 0; aleft = p;
                        if (kComp) rest = comp_drop(rest, G);
                        segment_costs();
                    }
                    const uint64_t on = ballot64(active);
                    if ((on & gmask) == 0) have = false;
                    if (on == 0 || __builtin_popcountll(ballot64(!have && !exhausted)) >= kFetchGroups * G) break;
                }
            }
        };
        if (ballot64(active) != 0) {
            if (ballot64(have && in_slot) != 0) steps(BoolConst<true>()); else steps(BoolConst<false>());
        }

        // ---------------------------------------------------------------- a group in which no lane moves will never move again
        const bool stuck = have && (ballot64(moved) & gmask) == 0;
        if (ballot64(stuck) != 0) {
            PRS_KEEP_BRANCH();
            if (stuck) {
                if (in_slot || slot_runs == 0) {                            // cannot happen (see above): give it up rather than wait for ever
                    if (gl == 0) {
                        if (times.cfg_status) times.cfg_status[ci] = PRS_CFG_STALLED;
                        if (times.greedy) static_cast<T *>(times.greedy)[ci] = CostTraits<T>::bad();
                    }
                    have = active = false; left = 0;
                } else {
                    in_slot = true;
                    own = slot_ring<kPacked>(lane, slot_runs); in = slot_ring<kPacked>(prod, slot_runs);
                    start_configuration(BoolConst<true>());
                }
            }
        }
    }
}

// One launch for all machines of a ring size: every wavefront works through the classes from the heaviest
// configurations (largest groups) to the lightest, so the long-running ones start first and the light
// ones fill the machine around them.
template <typename T, bool kComp, bool kSmall>
__global__ __launch_bounds__(kWave) void uni_times_kernel(RingShape shape, ConfigArrays cfg, int32_t p_max, int32_t q_max, int model,
                                                          TimesOut times, PlanHeader *plan, const int32_t *order, char *slots,
                                                          size_t slot_bytes, int32_t slot_runs, bool help)
{
    // LDS is addressed from 0: the kernel has no other LDS than what the launch asks for (no private array indexed by a variable, which the
    // compiler would move there)
    if (kSmall) shape = RingShape{SmallRings<kComp>::kRuns, SmallRings<kComp>::kRing};
    constexpr int kFirst = kSmall ? 0 : kLargeClass;
    char *slot = slots + static_cast<size_t>(blockIdx.x) * slot_bytes;
    uni_times_body<T, 64, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + kClasses - 1, kGiantPart, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 32, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + kClasses - 1, kRestPart, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 16, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + 4, kWholeClass, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 8, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + 3, kWholeClass, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 4, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + 2, kWholeClass, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 2, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + 1, kWholeClass, slot, slot_runs);
    __syncthreads();
    uni_times_body<T, 1, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kFirst + 0, kWholeClass, slot, slot_runs);
    if (!kSmall && help) {
        // while the last of the large machines run, wavefronts that have none begin with the heavy small ones
        __syncthreads();
        uni_times_body<T, 64, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kClasses - 1, kGiantPart, slot, slot_runs, true);
        __syncthreads();
        uni_times_body<T, 32, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, kClasses - 1, kRestPart, slot, slot_runs, true);
        __syncthreads();
        uni_times_body<T, 16, kComp, kSmall>(shape, cfg, p_max, q_max, model, times, plan, order, 4, kWholeClass, slot, slot_runs, true);
    }
}

template <typename T, bool kComp>
static void launch_uni_times_as(const UniLaunch &L)
{
    const RingShape shape = large_rings(L.p_max);
    if (L.cls < kLargeClass)
        hipLaunchKernelGGL((uni_times_kernel<T, kComp, true>), dim3(L.grid), dim3(kWave), L.lds_bytes, L.stream, shape, L.cfg, L.p_max,
                           L.q_max, L.model, L.times, L.plan, L.order, L.slots, L.slot_bytes, L.slot_p, L.help);
    else
        hipLaunchKernelGGL((uni_times_kernel<T, kComp, false>), dim3(L.grid), dim3(kWave), L.lds_bytes, L.stream, shape, L.cfg, L.p_max,
                           L.q_max, L.model, L.times, L.plan, L.order, L.slots, L.slot_bytes, L.slot_p, L.help);
}

hipError_t launch_uni_times(const UniLaunch &L)
{
    const bool comp = L.cfg.comp_m > 0;
    if (L.cost == PRS_COST_I64) {
        if (comp) launch_uni_times_as<int64_t, true>(L); else launch_uni_times_as<int64_t, false>(L);
    } else {
        if (comp) launch_uni_times_as<double, true>(L); else launch_uni_times_as<double, false>(L);
    }
    return hipGetLastError();
}

}  // namespace prs
