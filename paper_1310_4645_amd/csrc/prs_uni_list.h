// Uni-greedy schedules (Lowery & Langou, Algorithm 1, Section 5) of machines of up to 1024 processors on gfx950: the segment
// pipeline of the completion-time kernel on linked lists of processors.  Emits the pairs of every segment in the order of
// Algorithm 1 (ties by processor index, the root never sending) with their start times.
//
// At any time a processor is in exactly one place: in the stream that leaves a segment, waiting for the next one, or among
// the receivers (B) that go back into its segment.  A configuration therefore needs one ready time and one link per processor,
// 10 bytes of LDS, for all its streams and all B together, and nothing of them lies in global memory (rings of 32 entries per
// lane backed by the workspace, which larger machines still use, wrote and read 83 bytes a pair there and waited for them half of
// the time).  A configuration is run by G lanes (1 to 32); lane l runs segments l, l + G, ... and reads the stream of the lane
// before it (lane 0 that of the last lane, a round behind).  The first segment needs no pipeline: its pairs and its stream have a closed
// form (ListRound), which the lanes of the group write side by side when they take a machine.
//
// One iteration of a lane forms one pair from the two smallest keys (ready time, index) among the heads of its input stream A and
// of B.  The sender joins the running group of the lane's stream, the senders with the newest value: sorted by index, not yet
// readable.  A pair with a later value, or the end of the segment, closes the group and publishes it.  The value of the running
// group is a lower bound of everything that follows, so a reader that has taken all that is published may still use B below it.
//
// How the reader finds the head of A.  It keeps the next processor in a register and reads the one after it from the link.  The
// link of the last published processor does not exist yet when the reader takes it, and the reader then links that processor
// elsewhere.  So a publication is announced in registers (its first processor and how many they are) and the link from the
// processor published before it is only written if the reader had not taken that one when the iteration began; a reader that
// has taken exactly what was there before the last publication starts at the announced processor, others follow the link.  If
// the reader takes that processor in the very iteration in which the link is written, the write comes first in program order.
//
// The heads' successors and the neighbours' counters are asked for in the middle of a step, when publications and B are up to date;
// the pair is staged and the sender joins its group while they come.
//
// Pairs are staged in LDS, eight per lane (blocks of 8 of the output arrays), and leave side by side: a store instruction of 64
// separate 16-byte rows costs a CU's store path 10 to 12 cycles a row, rows of 64 bytes written by four lanes 3 cycles per 16 bytes.
// Segment numbers are runs of p - 1 equal ones; wavefronts that have nothing else left write them.
//
// What bounds it: the latency of a step, about 240 instructions that depend on each other in 0.7 us, at six wavefronts per CU, which is what
// the LDS holds; 3072 machines at once take hardly longer than 512.  Measured (rings -> lists): 100,000 machines of up to 1024 processors
// 51.6 -> 22.4 ms, 27,320 of up to 826 processors and 93 segments 19.8 -> 6.6, one machine of 256 and 64 segments 2.35 -> 1.57.  The sweep
// in steps: first version 46.0; selects and dummy writes instead of branches 31.7; four steps between two looks for finished blocks
// 29.5; fewer pairs per lane in the classes of few lanes 26.5; two machines of 1024 processors to a wavefront 23.9; first segments in closed
// form 22.4.  Few segments (rings, lists as they were, now): 20,000 machines of 1024 processors and two segments 10.6, 14.6, 5.8 ms;
// 100,000 of 31 and two 203, 391, 170 us; 100,000 of 2 and one 65, 260, 52 us.  Not taken: idle groups that help with the class below (33.7: its machines run on lanes that wait), wave priorities by size (no change), tickets drawn
// several at a time (no change).
#pragma once

#include "prs_device.h"
#include "prs_launch.h"

namespace prs {

constexpr int kStageL = 8;                                   // pairs of a block of the output that a lane collects
constexpr int kFlushL = 8;                                   // blocks a pass of the flush writes, eight lanes each
constexpr int kDescL = 32;                                   // blocks listed at a time
constexpr int kStepsL = 4;                                   // steps between two looks for finished blocks and configurations
constexpr int kSharedL = 4096;                               // pairs a wavefront, on average, up to which machines are shared out without tickets
constexpr int kFewL = 32;                                    // pairs of a machine up to which one lane writes its segment numbers
constexpr int kLookL = 64;                                   // such looks between two looks for groups that do not move

// LDS of a wavefront: room for `procs` processors per lane.  A processor goes by the address of its link.
struct ListLds {
    int32_t x;                  // links, 16 bits, begin at 0; the ready time of the processor that a link names is at x + 4 * (address of the link)
    int32_t times, pairs;       // staged start times [64][8]; their senders and receivers, 16 bits each [64][8]
    int32_t blocks;             // blocks to write [kDescL]; between the flushes links that nobody reads
    static __host__ __device__ __forceinline__ int32_t bytes(int32_t procs) { return kWave * procs * 10 + kWave * kStageL * 12 + kDescL * 8; }
    __device__ __forceinline__ explicit ListLds(int32_t procs)
    {
        x = kWave * procs * 2;
        times = x + kWave * procs * 8;
        pairs = times + kWave * kStageL * 8;
        blocks = pairs + kWave * kStageL * 4;
    }
};
static_assert(kDescL * 8 >= kWave * 2, "a link for every lane");

typedef uint32_t __attribute__((ext_vector_type(4), may_alias)) ListVec;           // staged pairs are written one by one
typedef uint32_t __attribute__((ext_vector_type(4), aligned(4), may_alias)) ListRow;   // rows of the output arrays
typedef uint32_t __attribute__((ext_vector_type(2), may_alias)) ListBlock;         // its place holds links between the flushes: none of them may move past it

// Lanes of a group are 64 / G (G = 32) or 16 / G lanes apart inside a row of 16, so that the lane before is one rotation away.
template <int G> struct ListLanes {
    static constexpr int kApart = G == 32 ? 2 : 16 / G;
    static __device__ __forceinline__ int in_group(int lane) { return G == 32 ? lane >> 1 : (lane & 15) / kApart; }
    static __device__ __forceinline__ int group(int lane) { return G == 32 ? lane & 1 : (lane >> 4) * kApart + (lane & (kApart - 1)); }
    static __device__ __forceinline__ int leader(int lane) { return G == 32 ? lane & 1 : (lane & 48) | (lane & (kApart - 1)); }
    static __device__ __forceinline__ uint64_t mask(int lane)
    {
        if (G == 32) return UINT64_C(0x5555555555555555) << (lane & 1);
        uint64_t m = 0;
        for (int i = 0; i < G; ++i) m |= UINT64_C(1) << (i * kApart);
        return m << leader(lane);
    }
    static __device__ __forceinline__ int previous(int v)
    {
        if (G == 1) return v;
        if (G == 32) return dpp_from<kDppWaveRor1>(dpp_from<kDppWaveRor1>(v));
        return dpp_from<kDppRowRor + (G == 1 ? 1 : kApart)>(v);
    }
    static __device__ __forceinline__ int next(int v)
    {
        if (G == 1) return v;
        if (G == 32) return dpp_from<kDppWaveRol1>(dpp_from<kDppWaveRol1>(v));
        return dpp_from<kDppRowRor + (G == 1 ? 1 : 16 - kApart)>(v);
    }
    template <typename T> static __device__ __forceinline__ T previous_value(T v)
    {
        int32_t w[2];
        __builtin_memcpy(w, &v, 8);
        w[0] = previous(w[0]); w[1] = previous(w[1]);
        __builtin_memcpy(&v, w, 8);
        return v;
    }
};

// What a lane does in a pass of the flush: eight lanes write a block, two its senders, two its receivers, four its start times.
struct ListRole {
    char *out;                  // where element `first` of block 0 goes; null: nowhere
    int32_t lds;                // where that of lane 0 is staged
    int shift;                  // log2 of the bytes of a lane's staged values; of a block in the output array
    int first, per_word;        // first element of a block that it writes; log2 of the 32-bit words of an element
    int half;                   // 0: senders, 16: receivers
    __device__ __forceinline__ ListRole(const SchedOut &s, const ListLds &at, int lane)
    {
        const int part = lane & 7;
        per_word = part >= 4 ? 1 : 0;
        first = per_word ? (part & 3) * 2 : (part & 1) * 4;
        shift = per_word ? 6 : 5;
        half = part < 2 ? 0 : 16;
        char *const base = per_word ? static_cast<char *>(s.tstart) : reinterpret_cast<char *>(part < 2 ? s.src : s.dst);
        out = base ? base + (first << (2 + per_word)) : nullptr;
        lds = (per_word ? at.times : at.pairs) + (first << (2 + per_word));
    }
};

// Writes the finished blocks of the lanes with `pend`: up to pair `last` of the output, from place `lo` of its block on.
__device__ __forceinline__ void list_flush(const ListRole &role, const ListLds &lds, int lane, uint64_t ready, bool pend, int64_t last, int lo)
{
    const int rank = rank_below(ready), total = __builtin_popcountll(ready);
    for (int from = 0; from < total; from += kDescL) {
        if (pend && rank >= from && rank < from + kDescL) {
            const uint64_t d = (static_cast<uint64_t>(last >> 3) << 12) | static_cast<uint32_t>(lane << 6 | lo << 3 | (static_cast<int>(last) & 7));
            *lds_at<ListBlock>(lds.blocks + (rank - from) * 8) = ListBlock{static_cast<uint32_t>(d), static_cast<uint32_t>(d >> 32)};
        }
        __builtin_amdgcn_wave_barrier();                                   // other lanes read what this one wrote
        const int n = total - from < kDescL ? total - from : kDescL;
        for (int i0 = 0; i0 < n; i0 += kFlushL) {
            const int i = i0 + (lane >> 3);
            const ListBlock listed = *lds_at<ListBlock>(lds.blocks + i * 8);
            const uint64_t d = static_cast<uint64_t>(listed[1]) << 32 | listed[0];
            const int bits = static_cast<int>(listed[0]), owner = (bits >> 6) & 63, from_e = (bits >> 3) & 7, to_e = bits & 7;
            const ListVec staged = *lds_at<ListVec>(role.lds + (owner << role.shift));
            ListRow v;
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = role.per_word ? staged[b] : __builtin_amdgcn_ubfe(staged[b], role.half, 16);
            char *const out = role.out + (static_cast<int64_t>(d >> 12) << role.shift);
            const bool mine = i < n && role.out != nullptr;
            const int end = role.first + (role.per_word ? 1 : 3);
            const bool full = mine && from_e <= role.first && end <= to_e;
            if (full) *reinterpret_cast<ListRow *>(out) = v;
            const bool part = mine && !full && role.first <= to_e && from_e <= end;
            if (ballot64(part) != 0) {
                PRS_KEEP_BRANCH();
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int e = role.first + (b >> role.per_word);
                    if (part && from_e <= e && e <= to_e) reinterpret_cast<uint32_t *>(out)[b] = v[b];
                }
            }
        }
    }
}

// The first segment, from time 0, goes in rounds: the processors that are left pair up with their neighbours, all at one time, and
// receivers are left.  Their list at the beginning of a round is
//     [extra] 0 first first+step first+2step ...      (count processors in all)
// where `extra`, if there is one, is the last processor of the round before, which found no partner: it is ready earlier and so
// comes first, and its index is the largest.  The root never sends (Lemma 1 (ii)).  All start times differ from round to round (tcomm > 0
// and no sum is smaller than its terms), so no order but this one can arise.
struct ListRound {
    int first, step, count, extra;             // extra -1: none
    __device__ __forceinline__ int pairs() const { return count >> 1; }
    // Pair e of the round: the processor that sends and the one that receives and is left.
    __device__ __forceinline__ void pair(int e, int &snd, int &rcv) const
    {
        const int at = first + (2 * e - (extra >= 0 ? 2 : 1)) * step;                // for e > 0: the neighbours at, at + step
        snd = e > 0 ? at : (extra >= 0 ? extra : first);
        rcv = e > 0 ? at + step : 0;
    }
    // Senders by index: place i of the round's part of the stream (the extra one comes last).
    __device__ __forceinline__ int sender(int i) const
    {
        if (extra >= 0) return i == pairs() - 1 ? extra : first + 2 * i * step;
        return i > 0 ? first + (2 * i - 1) * step : first;
    }
    __device__ __forceinline__ void next()
    {
        const int regular = count - (extra >= 0 ? 1 : 0), last = regular > 1 ? first + (regular - 2) * step : 0;   // of the list
        const int alone = (count & 1) != 0 ? last : -1;
        first += extra >= 0 ? step : 2 * step;
        step *= 2;
        count = pairs() + (count & 1);
        extra = alone;
    }
};

// With `help` a wavefront takes machines only while large ones (prs_uni_sched.hip) are not done.
template <typename T, int G>
__device__ __forceinline__ void uni_list_body(const ListLds &lds, int32_t procs, const ConfigArrays &cfg, int64_t n, int32_t p_max, int32_t q_max, const SchedOut &sched,
                                              PlanHeader *plan, const int32_t *order, int cls, bool roomy, bool &first, bool help)
{
    typedef ListLanes<G> Lanes;
    constexpr int kGroups = kWave / G;
    const int32_t count = plan->class_count[cls], begin = plan->class_begin[cls];
    if (count == 0) return;
    // nothing is left of a class that wavefronts have begun before
    if (!first && __hip_atomic_load(&plan->ticket[cls], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= static_cast<unsigned long long>(count)) return;
    // Tickets come from one address for the whole chip, which serves a wavefront about every 20 ns.  All wavefronts come to the first
    // class that has machines at one time: there each group has its first ticket without asking, and all of its tickets if these are
    // all or the machines are small.  A wavefront that has seen the end of a class asks no more.
    // First tickets go to one group of every wavefront before the next group has one if that leaves the other classes their wavefronts
    // or most machines are of this class, otherwise to wavefront by wavefront (20,000 machines of up to 64 processors and 24 segments, us: 327
    // and 382; 60,000 of up to 64 and 64: 1025 and 776).
    const uint32_t at_once = gridDim.x * kGroups;
    const bool shared = first && (static_cast<uint32_t>(count) <= at_once || sched.pair_capacity / gridDim.x <= kSharedL);
    bool given = first, over = false;
    const int lane = lane_id(), gl = Lanes::in_group(lane), leader = Lanes::leader(lane);
    const uint64_t gmask = Lanes::mask(lane);
    // the next ticket that the group has without asking, or the first one that is asked for
    uint32_t mine = !first ? 0 : roomy || count >= n / 2 ? Lanes::group(lane) * gridDim.x + blockIdx.x : Lanes::group(lane) + blockIdx.x * kGroups;
    first = false;
    const ListRole role(sched, lds, lane);
    const int32_t root = Lanes::group(lane) * (G * 2) * procs;         // link of processor 0 of the group's machine
    const int32_t unread = lds.blocks + lane * 2, stage_t = lds.times + lane * (kStageL * 8), stage_i = lds.pairs + lane * (kStageL * 4);
    auto X = [&](int32_t link) { return lds_at<T>(link * 4 + lds.x); };
    auto N = [&](int32_t link) { return lds_at<uint16_t>(link); };
    T huge = 0;                                                                     // above every time of a schedule
    huge = or_absent<T>(false, huge);

    // ---- per-group state (the same in all lanes of a group)
    bool have = false, exhausted = false;
    int64_t ci = 0, out_base = 0;
    int p = 2, q = 1;
    T c_full = 0, g_full = 0, c_last = 0, g_last = 0;
    // ---- per-lane state.  Positions count entries of a stream from the start of the configuration, p to a segment.
    int k = 0, left = 0;                // my segment, pairs it still has to form
    int32_t orel = 0, seen = 0;         // the next pair's place in the output of the configuration; the same when it was last looked at
    int rounds = 0;
    int pub = 0;                        // entries of my stream published
    uint32_t news = root;               // the last publication: its first processor, and how many (upper half)
    T newsV = 0;                        // and its ready time
    int32_t tail = root;                   // last processor published
    int apos = 0, aleft = 0;            // entries of my input stream taken (the first segment's none); those still to be taken in this segment
    int32_t ah = root;                     // head of A
    T xa0 = 0;                          // its ready time
    int32_t gf = root, gt = root, gi = root, gs = root;   // running group: first, last, the one inserted last, the one after that
    int gn = 0;                         // how many
    T lastS = 0;                        // its value (-1 before the first pair of a segment)
    int32_t bh = root, bt = root, bp = root, bi = root;   // B: head, last, the one before the newest value, the one inserted last
    int bn = 0, brun = 0;               // unread entries of B; pairs that were left when its newest value came
    T xb0 = 0, lastB = 0;               // ready time of B's head; newest value
    T cc = 0, gg = 0;                   // costs of my segment
    bool pend = false;                  // a block of staged pairs waits to be written
    int32_t pend_rel = 0;
    int pend_lo = 0;

    // what a step reads of its neighbours and of the lists, asked for half a step ahead
    int ahead = 0, reader = 0;          // entries published and not taken of the stream I read; entries taken of mine
    T plast = 0;                        // running value of my producer
    int32_t a1 = root, b1 = root;             // the processors after the heads
    T xa1 = 0, xb1 = 0;                 // and their ready times
    auto refresh = [&]() {
        __builtin_amdgcn_wave_barrier();
        ahead = Lanes::previous(pub) - apos;
        const uint32_t pnews = static_cast<uint32_t>(Lanes::previous(static_cast<int>(news)));
        const T pnewsV = Lanes::previous_value(newsV);
        plast = Lanes::previous_value(lastS);
        reader = Lanes::next(apos);
        const bool jump = ahead == static_cast<int>(pnews >> 16);
        ah = jump ? static_cast<int32_t>(pnews & 0xFFFF) : ah;
        xa0 = jump ? pnewsV : xa0;
        a1 = *N(ah); xa1 = *X(ah);
        b1 = *N(bh); xb1 = *X(bh);
    };

    // A walk behind a processor whose index is smaller ends at the last one of its value, which is larger.  If it does not, the list is
    // no list any more; the walk is bounded and the machine marked.  (The mark goes straight to memory: one that travels in a register
    // costs 2 % of the call, schedule_uni_100k 24.9 -> 25.4 ms.)
    auto out_of_order = [&]() { if (sched.cfg_status) sched.cfg_status[ci] = PRS_CFG_STALLED; };

    for (;;) {
        // ---------------------------------------------------------------- finished blocks leave
        const uint64_t ready = ballot64(pend);
        if (ready != 0) list_flush(role, lds, lane, ready, pend, out_base + pend_rel, pend_lo);
        pend = false;
        // ---------------------------------------------------------------- fetch a configuration
        if (have && (ballot64(k < q) & gmask) == 0) have = false;             // every lane of the group is through
        if ((++rounds & (kLookL - 1)) == 0) {
            PRS_KEEP_BRANCH();
            // The lane of the first segment that is not done never waits for another one: a group forms a pair in every round of steps.
            // One that formed none since the last look cannot go on; it is given up rather than waited for.  (Looked at in every round: 26.3 ms.)
            const uint64_t moved = ballot64(orel != seen);
            seen = orel;
            if (have && (moved & gmask) == 0) {
                if (gl == 0) {
                    if (sched.cfg_status) sched.cfg_status[ci] = PRS_CFG_STALLED;
                    if (sched.T_greedy) static_cast<T *>(sched.T_greedy)[ci] = CostTraits<T>::bad();
                }
                have = false; left = 0;
            }
        }
        if (ballot64(!have && !exhausted) != 0) {
            if (help && __hip_atomic_load(&plan->large_left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) exhausted = exhausted || !have;
            int64_t ticket = over ? count : mine;
            if (!given && !over) {
                const unsigned long long got = atomicAdd(&plan->ticket[cls], !have && !exhausted && gl == 0 ? 1ULL : 0ULL);
                const uint32_t l32 = __shfl(static_cast<uint32_t>(got), leader), h32 = __shfl(static_cast<uint32_t>(got >> 32), leader);
                ticket += static_cast<int64_t>((static_cast<uint64_t>(h32) << 32) | l32);
            }
            if (!have && !exhausted) {
                left = 0;
                if (given) mine = shared ? mine + at_once : at_once;
                if (ticket >= count) {
                    exhausted = true;
                } else {
                    ci = order[begin + ticket];
                    const Config<T> c = decode_config<T>(cfg, ci, p_max, q_max);
                    int32_t status = c.status;
                    if (status == PRS_CFG_OK) {
                        out_base = sched.pair_offset[ci];
                        const int64_t n_pairs = static_cast<int64_t>(c.p - 1) * c.q;
                        if (out_base < 0 || out_base + n_pairs > sched.pair_capacity) status = PRS_CFG_TOO_LARGE;
                    }
                    if (gl == 0) {
                        if (sched.cfg_status) sched.cfg_status[ci] = status;
                        if (status != PRS_CFG_OK && sched.T_greedy) static_cast<T *>(sched.T_greedy)[ci] = CostTraits<T>::bad();
                    }
                    if (status == PRS_CFG_OK) {
                        have = true;
                        p = c.p; q = c.q;
                        c_full = c.c_full; g_full = c.g_full; c_last = c.c_last; g_last = c.g_last;
                        k = gl; pub = 0; news = root; seen = -1;
                        tail = root;
                        apos = 0; aleft = p;
                        ah = bh = bt = gf = gt = gi = gs = root; a1 = b1 = root; xa0 = 0; newsV = 0;
                        gn = 0; lastS = T(-1); bn = 0;
                        const T c0 = q == 1 ? c_last : c_full, g0 = q == 1 ? g_last : g_full;
                        ListRound round = {1, 1, p, -1};
                        int32_t from = root;                                 // first of the stream
                        T t = 0;
                        for (int done = 0; round.count > 1;) {
                            const int pairs = round.pairs();
                            const T tc = wrap_add<T>(t, c0), tr = wrap_add<T>(tc, g0);
                            const int64_t o = out_base + done;
                            // the root ends the stream, before the last sender if both are ready at one time
                            const bool final = round.count == 2, with = final && tr == tc;
                            ListRound after = round;
                            after.next();
                            const T tc1 = wrap_add<T>(tr, c0);
                            const bool root_next = after.count == 2 && wrap_add<T>(tc1, g0) == tc1;
                            const int32_t then = final || root_next ? root : root + 2 * after.sender(0);
                            if (done == 0) { from = with ? root : root + 2; newsV = with ? tr : tc; }
                            for (int e = gl; e < pairs; e += G) {
                                int snd, rcv;
                                round.pair(e, snd, rcv);
                                if (sched.src) sched.src[o + e] = snd;
                                if (sched.dst) sched.dst[o + e] = rcv;
                                if (sched.tstart) static_cast<T *>(sched.tstart)[o + e] = t;
                                const int32_t x = root + 2 * round.sender(e);
                                *X(x) = e + 1 < pairs ? tc : final ? tr : tc1;             // of the next one
                                *N(x) = static_cast<uint16_t>(e + 1 < pairs ? root + 2 * round.sender(e + 1) : then);
                            }
                            if (final && gl == 0) {
                                const int32_t x = root + 2 * round.sender(0);
                                *X(root) = tc;
                                *N(root) = static_cast<uint16_t>(with ? x : root);
                                tail = with ? x : root;
                            }
                            done += pairs;
                            t = tr;
                            round = after;
                        }
                        // the first lane is through with it, and its reader finds all of it published at once
                        if (gl == 0) {
                            if (q == 1 && sched.T_greedy) static_cast<T *>(sched.T_greedy)[ci] = t;
                            k = G; pub = p;
                            news = static_cast<uint32_t>(from) | static_cast<uint32_t>(p) << 16;
                        } else {
                            newsV = 0;
                        }
                        left = k < q ? p - 1 : 0; orel = k * (p - 1);
                        cc = k == q - 1 ? c_last : c_full; gg = k == q - 1 ? g_last : g_full;
                    }
                }
            }
            given = shared;
            over = !shared && (over || ballot64(exhausted) != 0);
            if (ballot64(have) == 0 && ballot64(!exhausted) == 0) break;
            if (ballot64(left > 0) == 0) continue;                      // machines of one segment are done
            refresh();
        }

#pragma unroll 1
        for (int step = 0; step < kStepsL; ++step) {
            // ------------------------------------------------------------ the two smallest keys of A and B
            const int32_t a0 = ah, b0 = bh;
            const int32_t a2 = *N(a1), b2 = *N(b1);                                // what comes after them, for the next step
            const T xa2 = *X(a1), xb2 = *X(b1);
            const bool complete = ahead >= aleft;
            const int avail = complete ? aleft : ahead;
            const T va0 = or_absent<T>(avail > 0, xa0), va1 = or_absent<T>(avail > 1, xa1);
            const T vb0 = or_absent<T>(bn > 0, xb0), vb1 = or_absent<T>(bn > 1, xb1);
            // entries not published yet are >= the running value of the producer
            const T front = complete ? huge : plast;
            const bool x = (va0 < vb0) | ((va0 == vb0) & (a0 < b0));               // the smallest is A's head
            const T ux = x ? va1 : va0, vx = x ? vb0 : vb1;                        // heads after removing it
            const int32_t ui = x ? a1 : a0, vi = x ? b0 : b1;
            const bool y = (ux < vx) | ((ux == vx) & (ui < vi));                   // the second smallest comes from A
            const int32_t e1 = x ? a0 : b0, e2 = y ? ui : vi;
            const T t = y ? ux : vx;
            const bool ok = (left > 0) & !pend & (t < front);
            const T tc = wrap_add<T>(t, cc), tr = wrap_add<T>(tc, gg);
            const bool isroot = e1 == root;                                        // the root never sends (Lemma 1 (ii))
            const int32_t snd = isroot ? e2 : e1, rcv = isroot ? e1 : e2;
            const bool fresh = !(tc == lastS);
            const bool closing = ok & fresh & (gn > 0);
            if (ok) {
                --left;
                // ---- consume
                const int dA = (x ? 1 : 0) + (y ? 1 : 0);
                apos += dA; aleft -= dA; bn += dA - 2;
                ah = x & y ? a2 : (x | y ? a1 : a0); xa0 = x & y ? xa2 : (x | y ? xa1 : xa0);
                bh = x & y ? b0 : (x | y ? b1 : b2); xb0 = x & y ? xb0 : (x | y ? xb1 : xb2);
                // ---- the group of an earlier value is published, and linked behind what was published before it
                if (closing & (reader < pub)) { *N(tail) = static_cast<uint16_t>(gf); *X(tail) = lastS; }
                __builtin_amdgcn_wave_barrier();                                   // before any of the links below
                tail = closing ? gt : tail; newsV = closing ? lastS : newsV;
                news = closing ? static_cast<uint32_t>(gf) | static_cast<uint32_t>(gn) << 16 : news;
                pub += closing ? gn : 0;
                lastS = tc;
                // ---- the receiver joins B
                const bool empty = bn == 0, same = !empty & (tr == lastB), late = same & (rcv < bt);
                if (ballot64(late) != 0) {                                         // not behind the others of the same ready time
                    PRS_KEEP_BRANCH();
                    if (late) {
                        const bool older = brun < left + bn;                       // the entry before the newest value is unread
                        int32_t before = bp, after = older ? static_cast<int32_t>(*N(bp)) : bh;
                        bool head = !older;
                        if (after < rcv) {
                            before = brun <= left + bn && bi < rcv ? bi : after;
                            after = *N(before);
                            for (int w = 0; after < rcv && w < kUniListProcs; ++w) { before = after; after = *N(before); }
                            if (after < rcv) out_of_order();
                            head = false;
                        }
                        *N(rcv) = static_cast<uint16_t>(after); *X(rcv) = tr;
                        if (head) { bh = rcv; xb0 = tr; } else { *N(before) = static_cast<uint16_t>(rcv); }
                    }
                }
                if (!(empty | late)) { *N(bt) = static_cast<uint16_t>(rcv); *X(bt) = tr; }
                bh = empty ? rcv : bh; xb0 = empty ? tr : xb0;
                bp = same ? bp : bt; brun = same ? brun : left;
                bt = late ? bt : rcv; bi = rcv;
                lastB = tr;
                ++bn;
            }
            refresh();
            if (ok) {
                // ---- stage the pair
                const int at = (static_cast<int>(out_base) + orel) & (kStageL - 1);
                *lds_at<T>(stage_t + at * 8) = t;
                *lds_at<uint32_t>(stage_i + at * 4) = static_cast<uint32_t>((snd - root) | (rcv - root) << 16) >> 1;
                if (at == kStageL - 1 || left == 0) {
                    const int first = at + 1 - (p - 1 - left);                     // place of the segment's first pair if it is in this block
                    pend = true; pend_rel = orel; pend_lo = first > 0 ? first : 0;
                }
                ++orel;
                // ---- the sender joins the running group
                const bool append = fresh | (snd > gt), front_of = fresh | (snd < gf);
                int32_t pred = append ? gt : gi, succ = front_of ? gf : gs;
                const bool behind = append | front_of | ((gi < snd) & (snd < gs));
                if (ballot64(!behind) != 0) {
                    PRS_KEEP_BRANCH();
                    if (!behind) {                                                 // neither end nor behind the one inserted last
                        pred = snd > gi ? gi : gf;
                        succ = *N(pred);
                        for (int w = 0; succ < snd && w < kUniListProcs; ++w) { pred = succ; succ = *N(pred); }
                        if (succ < snd) out_of_order();
                    }
                }
                *N(front_of ? unread : pred) = static_cast<uint16_t>(snd);
                *N(snd) = static_cast<uint16_t>(succ);
                *X(snd) = tc;                                                      // the processor after it has the same
                gf = front_of ? snd : gf; gt = append ? snd : gt;
                gi = snd; gs = succ;
                gn = fresh ? 1 : gn + 1;
            }
            // ------------------------------------------------------------ end of a segment: the root's final state closes its stream
            const bool ending = ok & (left == 0);
            if (ballot64(ending) != 0) {
                PRS_KEEP_BRANCH();
                if (ending) {
                    const bool with = lastB == lastS;                              // the root joins the running group, in front
                    if (with) { *N(root) = static_cast<uint16_t>(gf); *X(root) = lastS; gf = root; }
                    else { *N(gt) = static_cast<uint16_t>(root); *X(gt) = lastB; gt = root; }
                    ++gn;
                    if (closing | (reader < pub)) { *N(tail) = static_cast<uint16_t>(gf); *X(tail) = lastS; }
                    news = closing ? news + (static_cast<uint32_t>(gn) << 16) : static_cast<uint32_t>(gf) | static_cast<uint32_t>(gn) << 16;
                    newsV = closing ? newsV : lastS;
                    pub += gn; tail = gt;
                    if (k == q - 1 && sched.T_greedy) static_cast<T *>(sched.T_greedy)[ci] = lastB;
                    k += G; orel += (G - 1) * (p - 1);
                    left = k < q ? p - 1 : 0; aleft = p;
                    gn = 0; lastS = T(-1); bn = 0;
                    cc = k == q - 1 ? c_last : c_full; gg = k == q - 1 ? g_last : g_full;
                }
                refresh();
            }
        }
    }
}

// Every wavefront works through the classes from the heaviest configurations (largest groups) to the lightest.  `begun`: others may have
// taken tickets already.
template <typename T>
__device__ __forceinline__ void uni_list_all(int32_t procs, const ConfigArrays &cfg, int64_t n, int32_t p_max, int32_t q_max, const SchedOut &sched,
                                             PlanHeader *plan, const int32_t *order, bool begun, bool help)
{
    // LDS is addressed from 0: the kernel has no other LDS than what the launch asks for.  Private arrays that are indexed by a variable
    // would change that: the compiler moves them to LDS, to address 0.
    const ListLds lds(procs);
    // Lanes without a machine read and follow the links of their place like all others (refresh): every link names a processor of the
    // wavefront from the start, whatever the LDS held before.
    for (int32_t at = lane_id() * 16; at < ListLds::bytes(procs); at += kWave * 16) *lds_at<ListVec>(at) = ListVec{0, 0, 0, 0};
    __syncthreads();
    int64_t wanted = 0;                                                    // wavefronts that hold the whole batch
    for (int k = 0; k < kClasses; ++k) wanted += plan->class_count[k] >> (kClasses - k);
    const bool roomy = wanted <= gridDim.x;
    bool first = !begun;
    uni_list_body<T, 32>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 5, roomy, first, help);
    __syncthreads();
    uni_list_body<T, 16>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 4, roomy, first, help);
    __syncthreads();
    uni_list_body<T, 8>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 3, roomy, first, help);
    __syncthreads();
    uni_list_body<T, 4>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 2, roomy, first, help);
    __syncthreads();
    uni_list_body<T, 2>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 1, roomy, first, help);
    __syncthreads();
    uni_list_body<T, 1>(lds, procs, cfg, n, p_max, q_max, sched, plan, order, 0, roomy, first, help);
    __syncthreads();
}

}  // namespace prs
