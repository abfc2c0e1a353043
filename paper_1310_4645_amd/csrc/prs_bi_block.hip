// Bi-greedy schedules (Lowery & Langou, Algorithm 2, Section 6.2) for machines of thousands of processors on
// gfx950: one block of eight wavefronts per configuration, or one of its wavefronts.
//
// Every list of Algorithm 2 is a bit set over the processors, list lengths are population counts, "first k entries" a
// rank select inside a word, list positions prefix sums.  run_bi_wide keeps the sets in registers and the running transfers in a
// list; run_bi_block, which keeps times per processor in the workspace slot, does what does not fit there: more than 64
// transfers running at once.
//
// What bounds it: the chain of visits of the longest configuration, 24 a segment, three quarters of which pair somebody, at 4600
// cycles each on eight wavefronts: sums inside and between the wavefronts, and 400 instructions that depend on each
// other.  On one wavefront a visit needs neither a barrier nor a sum over the block, so machines of up to 16384 processors (four
// words of every set per lane; with six or eight the registers spill, 12.6 -> 17.4 and 28.6 ms on 16 of up to 22,709) run on one: 19 of
// up to 5006 processors and 495 segments 14.6 -> 7.5 ms, 26 of up to 2223 4.76 -> 2.23.  Schedules, whose indices one wavefront writes more slowly than eight,
// go to one up to 4096 processors only (16 machines of 16,384 and 64 segments 4.0 ms on eight wavefronts, 9.4 on one; of 8000 4.4 and 5.8).  64 machines of 1024 to 65536 processors, completion
// times: 263 ms with times per processor (about 14 barriers a visit, scattered updates of S, R and C1, all of them read
// again at every event), 41.0 with two sums over the block and a loop over the wavefronts' parts, 38.8 so.  Measured and not
// taken: what a visit writes held back until the next one has its row (no change), eight entries of the list at a time
// (41.0), four wavefronts with four words per thread (44.7).
#include "prs_device.h"
#include "prs_launch.h"

namespace prs {

constexpr int kBlockThreads = 512;
constexpr int kBlockWaves = kBlockThreads / kWave;

__host__ __device__ inline size_t bb_align(size_t v) { return (v + 255) / 256 * 256; }

// workspace slot of a block: S, R, C1 (8 B per processor), flags and count of sent segments (4 B), the two pairing
// lists, the per-segment counters, the sent bitmap [q][W].  The 64 pairs of sets of run_bi_wide (16 B per processor) lie where
// run_bi_block, which begins from the start, keeps S, R and C1 (they fit from 126 processors on).
struct BlockSlot { size_t S, R, C1, nsent, sendList, recvList, rem, sent, sets, total; };

__host__ __device__ inline BlockSlot bi_block_slot(int32_t p_cap, int32_t q_cap)
{
    BlockSlot L;
    const size_t p = static_cast<size_t>(p_cap), q = static_cast<size_t>(q_cap), W = (p + 63) / 64;
    size_t o = 0;
    L.sets = o;
    L.S = o; o += bb_align(p * 8);
    L.R = o; o += bb_align(p * 8);
    L.C1 = o; o += bb_align(p * 8);
    L.nsent = o; o += bb_align(p * 4);
    L.sendList = o; o += bb_align((p / 2 + 1) * 4);
    L.recvList = o; o += bb_align((p / 2 + 1) * 4);
    L.rem = o; o += bb_align(q * 4);
    L.sent = o; o += bb_align(W * q * 8);
    L.total = o;
    return L;
}

size_t bi_block_slot_bytes(int32_t p_cap, int32_t q_cap) { return bi_block_slot(p_cap, q_cap).total; }
// LDS: 7 bit sets and 2 arrays of 16-bit list positions of Wcap words, then the scratch of the block-wide sums
size_t bi_block_lds_bytes(int32_t p_cap)
{
    const size_t W = (static_cast<size_t>(p_cap) + 63) / 64;
    return bb_align(W * 8 * 7) + bb_align(W * 2 * 2) + 1024;
}

// run_bi_block: the same sequence of set operations as the one-wavefront kernel, the words of the bit sets and the processors
// spread over the threads of the block: thread w owns the words w, w + 512, ... of every set, sums and prefix sums go
// through the wavefronts and then through LDS.  The bit sets of a visit sit in LDS (7 sets of up to about 1060 words), the
// per-processor times, the pairing lists, the per-segment counters and the sent bitmap in the block's workspace slot.
struct BlockScratch {
    int32_t *part;       // [3][kBlockWaves] partial sums of the wavefronts
    double *tpart;       // [kBlockWaves] partial minima (bit patterns of T)
};

// sums of three values over the block (the same result in every thread)
__device__ __forceinline__ void block_sum3(const BlockScratch &bs, int &a, int &b, int &c)
{
    const int lane = lane_id(), wave = static_cast<int>(threadIdx.x) >> 6;
    a = wave_sum(a); b = wave_sum(b); c = wave_sum(c);
    __syncthreads();                                             // earlier readers of the scratch are through
    if (lane == 0) { bs.part[wave] = a; bs.part[kBlockWaves + wave] = b; bs.part[2 * kBlockWaves + wave] = c; }
    __syncthreads();
    int sa = 0, sb = 0, sc = 0;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) { sa += bs.part[w]; sb += bs.part[kBlockWaves + w]; sc += bs.part[2 * kBlockWaves + w]; }
    a = sa; b = sb; c = sc;
}

// exclusive prefix sums of two values over the threads of the block, and their totals
__device__ __forceinline__ void block_scan2(const BlockScratch &bs, int a, int b, int &exA, int &exB, int &totA, int &totB)
{
    const int lane = lane_id(), wave = static_cast<int>(threadIdx.x) >> 6;
    const int incA = wave_inclusive_scan(a), incB = wave_inclusive_scan(b);
    __syncthreads();
    if (lane == kWave - 1) { bs.part[wave] = incA; bs.part[kBlockWaves + wave] = incB; }
    __syncthreads();
    int beforeA = 0, beforeB = 0, sa = 0, sb = 0;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) {
        const int va = bs.part[w], vb = bs.part[kBlockWaves + w];
        if (w < wave) { beforeA += va; beforeB += vb; }
        sa += va; sb += vb;
    }
    exA = beforeA + incA - a; exB = beforeB + incB - b;
    totA = sa; totB = sb;
}

template <typename T> __device__ __forceinline__ T block_min(const BlockScratch &bs, T v)
{
    const int lane = lane_id(), wave = static_cast<int>(threadIdx.x) >> 6;
    v = wave_min<T>(v);
    T *tp = reinterpret_cast<T *>(bs.tpart);
    __syncthreads();
    if (lane == 0) tp[wave] = v;
    __syncthreads();
    T m = tp[0];
#pragma unroll
    for (int w = 1; w < kBlockWaves; ++w) { const T u = tp[w]; m = u < m ? u : m; }
    return m;
}

template <typename T, bool kSched>
__device__ T run_bi_block(const Config<T> &c, char *lds, char *slot, const BlockSlot &sl, int Wc, const SchedOut &sched,
                          int64_t out_base, int32_t *status)
{
    const int tid = static_cast<int>(threadIdx.x), lane = lane_id(), wave = tid >> 6;
    const int p = c.p, q = c.q;
    const int W = (p + 63) >> 6;
    T *S = reinterpret_cast<T *>(slot + sl.S);
    T *R = reinterpret_cast<T *>(slot + sl.R);
    T *C1 = reinterpret_cast<T *>(slot + sl.C1);
    int32_t *nsent = reinterpret_cast<int32_t *>(slot + sl.nsent);
    int32_t *sendList = reinterpret_cast<int32_t *>(slot + sl.sendList);
    int32_t *recvList = reinterpret_cast<int32_t *>(slot + sl.recvList);
    int32_t *rem = reinterpret_cast<int32_t *>(slot + sl.rem);
    uint64_t *sent = reinterpret_cast<uint64_t *>(slot + sl.sent);           // [q][W]
    uint64_t *mk = reinterpret_cast<uint64_t *>(lds);
    uint64_t *sfree = mk, *rfree = mk + Wc, *compF = mk + 2 * Wc, *compL = mk + 3 * Wc;
    uint64_t *sendSet = mk + 4 * Wc, *recvSet = mk + 5 * Wc, *lateL = mk + 6 * Wc;
    // list positions of a word's first sender and receiver: below 2^16, a list has at most p/2 <= 32768 entries
    uint16_t *prefS = reinterpret_cast<uint16_t *>(lds + bb_align(static_cast<size_t>(Wc) * 8 * 7)), *prefR = prefS + Wc;
    BlockScratch bs;
    bs.part = reinterpret_cast<int32_t *>(lds + bb_align(static_cast<size_t>(Wc) * 8 * 7) + bb_align(static_cast<size_t>(Wc) * 2 * 2));
    bs.tpart = reinterpret_cast<double *>(bs.part + 3 * kBlockWaves + 16);
    // nsent[i] also carries the kind of i's latest transfers: bit 30 = it last sent the smaller last segment,
    // bit 29 = it last received it
    constexpr int32_t kSentShort = 1 << 30, kRecvShort = 1 << 29, kCount = kRecvShort - 1;
    const bool ragged = c.sz_last != c.sz, guardL = ragged && c.g_last > 0;

    for (int i = tid; i < p; i += kBlockThreads) { S[i] = 0; R[i] = 0; C1[i] = 0; nsent[i] = 0; }
    for (int j = tid; j < q; j += kBlockThreads) rem[j] = p - 1;
    for (int64_t k = tid; k < static_cast<int64_t>(q) * W; k += kBlockThreads) sent[k] = 0;
    __syncthreads();

    const T kInf = CostTraits<T>::inf();
    T t = 0, Tmax = 0;
    int ndone = 0, segStart = 0;
    int64_t emitted = 0;
    bool lateOnly = false;
    const int64_t max_events = 4 * static_cast<int64_t>(p) * q + 16;
    for (int64_t ev = 0;; ++ev) {
        if (ev > max_events) { *status = PRS_CFG_STALLED; return CostTraits<T>::bad(); }
        // ---- port and computation state of every processor at time t, as bit sets (wavefront v takes words v, v+8, ...)
        T minOld = kInf, minLate = kInf;             // next time a port frees / a processor may take in the last segment
        int cs = 0, cr = 0, cu = 0;                  // free send ports, free receive ports, processors with either
        int csAll = 0;                               // free send ports of processors with something left to send
        for (int w = wave; w < W; w += kBlockWaves) {
            const int i = w * kWave + lane;
            const bool in = i < p;
            const T s = in ? S[i] : 0, r = in ? R[i] : 0, c1 = in ? C1[i] : 0;
            const int32_t nsnt = in ? nsent[i] : 0;
            const bool live = in && (i == 0 || (nsnt & kCount) < q);   // still a member of some segment
            const bool sf = live && i != 0 && s <= t;              // the root never sends
            const bool rf = live && r <= t;
            const bool busy = in && c1 <= t && t < r;              // computing now
            const bool pend = in && t < c1;                        // computation scheduled ahead
            // A transfer begun now must not run into that computation.  It was scheduled before t: against a segment
            // of its own size that settles it; against the other size the rounded sums are compared.
            const bool rshort = (nsnt & kRecvShort) != 0;
            const bool cF = busy || (pend && (!rshort || t + c.c_full > c1));
            const bool cL = busy || (pend && (rshort || !ragged || t + c.c_last > c1));
            // Section 2 the other way round: the combine of the smaller last segment, received now, would begin while
            // this processor is still sending a full one; it becomes eligible at s - tcomm(last)
            const bool lt = in && guardL && !(nsnt & kSentShort) && s > t + c.c_last;
            if (in && s > t && s < minOld) minOld = s;
            if (in && r > t && r < minOld) minOld = r;
            if (lt) { const T v = s - c.c_last; if (v > t && v < minLate) minLate = v; }
            const uint64_t bsf = ballot64(sf), brf = ballot64(rf), bcF = ballot64(cF), bcL = ballot64(cL), blt = ballot64(lt);
            if (lane == 0) {
                sfree[w] = bsf; rfree[w] = brf; compF[w] = bcF; compL[w] = bcL; lateL[w] = blt;
                cs += __popcll(bsf & ~bcL);
                cr += __popcll(brf & ~bcL);
                cu += __popcll((bsf | brf) & ~bcL);
                csAll += __popcll(bsf);
            }
        }
        minOld = block_min<T>(bs, minOld);
        if (guardL) minLate = block_min<T>(bs, minLate);
        block_sum3(bs, cs, cr, cu);                   // also makes the bit sets visible to every thread
        { int z0 = 0, z1 = 0; block_sum3(bs, csAll, z0, z1); }
        T minNew = kInf, minNewLate = kInf;
        while (segStart < q && rem[segStart] == 0) ++segStart;
        // At a time at which no port frees the candidates of every segment but the last have only become fewer
        // since the event before: only the last segment is visited.
        for (int j = (lateOnly && segStart < q - 1) ? q - 1 : segStart; j < q; ++j) {
            // no further pair can form at this t: a pair needs a free send port and a free receive port on two
            // different processors
            if (cs == 0 || cr == 0 || cu < 2) break;
            int remj = rem[j];
            if (remj == 0) continue;                     // everybody has sent segment j
            const bool last = j == q - 1;
            const T cj = last ? c.c_last : c.c_full, gj = last ? c.g_last : c.g_full;
            // ---- pass A: the three lists of this visit as bit sets (thread w owns word w), and their lengths
            int ns_ = 0, nr_ = 0, nf_ = 0, cand_sent = 0;
            for (int w = tid; w < W; w += kBlockThreads) {
                uint64_t valid = ~UINT64_C(0);
                if (w == W - 1 && (p & 63)) valid = (UINT64_C(1) << (p & 63)) - 1;
                const uint64_t row = sent[static_cast<size_t>(j) * W + w];
                const uint64_t memb = ~row & valid;
                const uint64_t comp = last ? compL[w] : compF[w];
                const uint64_t sOK = memb & ~comp & sfree[w], rOK = memb & ~comp & rfree[w] & ~(last ? lateL[w] : UINT64_C(0));
                const uint64_t fr = sOK & rOK, so = sOK ^ fr, ro = rOK ^ fr;
                ns_ += __popcll(so); nr_ += __popcll(ro); nf_ += __popcll(fr);
                cand_sent += ((sfree[w] | rfree[w]) & ~comp & row & valid) != 0 ? 1 : 0;
            }
            block_sum3(bs, ns_, nr_, nf_);
            // ---- processors with both ports free go to the shorter list
            int toSendLast, toRecvFirst;
            if (ns_ == nr_) {
                toSendLast = toRecvFirst = nf_ / 2;
            } else if (ns_ < nr_) {
                const int y = nr_ - ns_, mm = nf_ < y ? nf_ : y, xx = (nf_ - mm) / 2;
                toSendLast = mm + xx; toRecvFirst = xx;
            } else {
                const int y = ns_ - nr_, mm = nf_ < y ? nf_ : y, xx = (nf_ - mm) / 2;
                toRecvFirst = mm + xx; toSendLast = xx;
            }
            const int sN = ns_ + toSendLast, rN = nr_ + toRecvFirst;
            const int l = sN < rN ? sN : rN;
            if (l == 0) {
                // nobody paired although no candidate had already sent j: the candidates of later segments are a
                // subset of these, so none of them can pair at this t either -- except the last segment, whose
                // shorter transfer is kept out by fewer pending computations
                int z0 = 0, z1 = 0;
                block_sum3(bs, cand_sent, z0, z1);
                if (cand_sent == 0) {
                    if (last) break;
                    j = q - 2;                               // go on with the last segment
                }
                continue;
            }
            // ---- pass B: final send and receive sets (first l of each), word by word with running ranks
            int carryF = 0, carryS = 0, carryR = 0, gone = 0;
            for (int w0 = 0; w0 < W; w0 += kBlockThreads) {
                const int w = w0 + tid;
                const bool on = w < W;
                uint64_t fr = 0, so = 0, ro = 0;                          // the three lists of pass A again (nothing has changed)
                if (on) {
                    uint64_t valid = ~UINT64_C(0);
                    if (w == W - 1 && (p & 63)) valid = (UINT64_C(1) << (p & 63)) - 1;
                    const uint64_t memb = ~sent[static_cast<size_t>(j) * W + w] & valid;
                    const uint64_t comp = last ? compL[w] : compF[w];
                    const uint64_t sOK = memb & ~comp & sfree[w], rOK = memb & ~comp & rfree[w] & ~(last ? lateL[w] : UINT64_C(0));
                    fr = sOK & rOK; so = sOK ^ fr; ro = rOK ^ fr;
                }
                const int pf = __popcll(fr);
                int exF, exDummy, totF, totDummy;
                block_scan2(bs, pf, 0, exF, exDummy, totF, totDummy);
                exF += carryF;                                            // free-list rank of this word's first entry
                const uint64_t frR = lowest_bits(fr, toRecvFirst - exF);
                const uint64_t frS = highest_bits(fr, exF + pf - (nf_ - toSendLast));
                uint64_t sset = so | frS, rset = ro | frR;
                const int ps = __popcll(sset), pr = __popcll(rset);
                int exS, exR, totS, totR;
                block_scan2(bs, ps, pr, exS, exR, totS, totR);
                exS += carryS; exR += carryR;
                sset = lowest_bits(sset, l - exS);
                rset = lowest_bits(rset, l - exR);
                if (on) {
                    sendSet[w] = sset; recvSet[w] = rset;
                    prefS[w] = static_cast<uint16_t>(exS < 65535 ? exS : 65535);       // words past the l-th entry hold nobody
                    prefR[w] = static_cast<uint16_t>(exR < 65535 ? exR : 65535);
                    sent[static_cast<size_t>(j) * W + w] |= sset;
                    const uint64_t sf0 = sfree[w], rf0 = rfree[w], open = ~compL[w];
                    sfree[w] = sf0 & ~sset;
                    rfree[w] = rf0 & ~rset;
                    gone += __popcll((sf0 | rf0) & open) - __popcll(((sf0 & ~sset) | (rf0 & ~rset)) & open);
                }
                carryF += totF; carryS += totS; carryR += totR;
            }
            __syncthreads();
            // ---- pass C: bit sets -> index lists in ascending processor order (a wavefront expands one word at a time,
            // only the words that hold a sender or a receiver)
            for (int w0 = wave * kWave; w0 < W; w0 += kBlockThreads) {
                const int wl = w0 + lane;
                uint64_t some = ballot64(wl < W && (sendSet[wl] | recvSet[wl]) != 0);
                while (some != 0) {
                    const int w = w0 + __builtin_ctzll(some);
                    some &= some - 1;
                    const uint64_t ss = sendSet[w], rs = recvSet[w];
                    if ((ss >> lane) & 1) sendList[prefS[w] + rank_below(ss)] = w * kWave + lane;
                    if ((rs >> lane) & 1) recvList[prefR[w] + rank_below(rs)] = w * kWave + lane;
                }
            }
            __threadfence_block();
            __syncthreads();
            // ---- pass D: entry-wise pairing
            const T tc = t + cj, tr = tc + gj;
            if (!(tc > t)) { *status = PRS_CFG_STALLED; return CostTraits<T>::bad(); }
            const bool shortNow = last && ragged;
            for (int e = tid; e < l; e += kBlockThreads) {
                const int32_t a = sendList[e], b = recvList[e];        // no processor is in both lists of a visit
                S[a] = tc;
                nsent[a] = (((nsent[a] & kCount) + 1) | (nsent[a] & kRecvShort)) | (shortNow ? kSentShort : 0);
                nsent[b] = (nsent[b] & ~kRecvShort) | (shortNow ? kRecvShort : 0);
                R[b] = tr;
                C1[b] = tc;
                if (kSched) {
                    const int64_t o = out_base + emitted + e;
                    if (sched.src) sched.src[o] = a;
                    if (sched.dst) sched.dst[o] = b;
                    if (sched.seg) sched.seg[o] = j;
                    if (sched.tstart) static_cast<T *>(sched.tstart)[o] = t;
                }
            }
            emitted += l;
            if (tc < minNew) minNew = tc;
            if (tr < minNew) minNew = tr;
            if (guardL && !last && tc > t + c.c_last) {           // these senders cannot take the last segment in yet
                for (int w = tid; w < W; w += kBlockThreads) lateL[w] |= sendSet[w];
                const T v = tc - c.c_last;
                if (v > t && v < minNewLate) minNewLate = v;
            }
            cs -= l; cr -= l; csAll -= l;
            int g0 = 0, g1 = 0;
            block_sum3(bs, gone, g0, g1);
            cu -= gone;
            remj -= l;
            if (tid == 0) rem[j] = remj;
            if (remj == 0) {                              // only the root is left: it finishes after the last arrival
                if (tr > Tmax) Tmax = tr;
                ++ndone;
            }
            __threadfence_block();
            __syncthreads();
        }
        if (ndone == q) break;
        T tn = minOld < minNew ? minOld : minNew;
        const T tl = minLate < minNewLate ? minLate : minNewLate;
        // without a free send port on a processor that still has something to send nothing can pair before a port frees
        lateOnly = csAll > 0 && tl < tn;
        if (lateOnly) tn = tl;
        if (!(tn < kInf)) { *status = PRS_CFG_STALLED; return CostTraits<T>::bad(); }
        t = tn;
        __threadfence_block();
        __syncthreads();                              // the pairs of this event are in S, R, C1 before the next state pass
    }
    return Tmax;
}

// ---- the usual path: sets in registers, running transfers as a list --------------------------------------------------
//
// Thread i owns the words i kw .. i kw + kw - 1 of every bit set, kw = 1, 2 or 3 (up to 4 on one wavefront), and keeps them in registers.  The
// kernel for three words serves batches whose bound passes 65536 processors (16 machines of 66,000, 8 segments: 14.6 ms on
// run_bi_block, 2.1 so; its registers cost machines of two words a sixth, 20 segments on 16 of 40,000 3.7 -> 4.3 ms).
// All pairs of a visit (time t, segment j) have the same end of send and end of combine, so the ports and computations
// of Algorithm 2 are a list of groups (end of send, end of combine, set of senders, set of receivers): lane e of EVERY
// wavefront holds the two times of entry e, the sets lie in the workspace slot, word by word written and read by the
// thread that owns the word.  Nothing is kept per processor, and a visit needs one sum over the block (the lengths of the
// three lists, the prefix counts of their parts and a few yes/no questions travel in 16 bytes per wavefront); a sum is
// one barrier, with two buffers in turn: a wavefront that writes a buffer again has passed the barrier of the sum in between,
// which nobody reaches before it has read the first.
// Processors that have sent everything stay in the sets: they hold no segment, so they never pair.
constexpr int kWideWords = 65536 / 64 / kBlockThreads;     // words per thread on machines of up to 65536 processors
constexpr int kWideProcs = kBlockThreads * kWideWords * 64;
constexpr int kAloneWords = 4, kAloneWordsSched = 1;       // words per lane up to which one wavefront runs a machine by itself
constexpr int kWideEntries = kWave;                        // running transfers, one per lane

template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_rows(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, ROWS == 0xF);
}
// inclusive prefix sum over the 64 lanes by moves inside the vector unit (row_shr 1, 2, 4, 8, then the last lane of a row
// of 16 to the next row and of the lower half to the upper half)
__device__ __forceinline__ int dpp_inclusive_scan(int v)
{
    v += dpp_rows<0x111, 0xF>(v);
    v += dpp_rows<0x112, 0xF>(v);
    v += dpp_rows<0x114, 0xF>(v);
    v += dpp_rows<0x118, 0xF>(v);
    v += dpp_rows<0x142, 0xA>(v);
    v += dpp_rows<0x143, 0xC>(v);
    return v;
}
// sum over the eight lanes of half a row: neighbours, pairs, the other quad
__device__ __forceinline__ int dpp_sum8(int v)
{
    v += dpp_rows<0xB1, 0xF>(v);
    v += dpp_rows<0x4E, 0xF>(v);
    v += dpp_rows<0x141, 0xF>(v);
    return v;
}
// lowest_bits where few lanes of a wavefront have to search, one in a list that all lanes hold words of: the whole wavefront looks
// at that lane's word, a bit to a lane.
__device__ __forceinline__ uint64_t lowest_bits_of_few(uint64_t mask, int k, int lane)
{
    const int n = __popcll(mask);
    uint64_t some = k > 0 ? mask : 0;
    uint64_t search = ballot64(k > 0 && k < n);
    while (search != 0) {
        const int who = __builtin_ctzll(search);
        search &= search - 1;
        const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(mask)), who),
                       hi = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(mask >> 32)), who);
        const uint64_t w = (static_cast<uint64_t>(hi) << 32) | lo;
        const int kk = __builtin_amdgcn_readlane(k, who);
        const uint64_t found = ballot64(rank_below(w) < kk) & w;
        some = lane == who ? found : some;
    }
    return some;
}
template <int CTRL, typename T> __device__ __forceinline__ T dpp_min(T v)
{
    int32_t w[2];
    __builtin_memcpy(w, &v, 8);
    w[0] = dpp_rows<CTRL, 0xF>(w[0]); w[1] = dpp_rows<CTRL, 0xF>(w[1]);
    T u;
    __builtin_memcpy(&u, w, 8);
    return u < v ? u : v;
}
// smallest value of the 64 lanes: rotations inside the rows of 16, then one lane of each row
template <typename T> __device__ __forceinline__ T wave_min_dpp(T v)
{
    v = dpp_min<0x128, T>(v); v = dpp_min<0x124, T>(v); v = dpp_min<0x122, T>(v); v = dpp_min<0x121, T>(v);
    int32_t w[2];
    __builtin_memcpy(w, &v, 8);
    T m = v;
#pragma unroll
    for (int r = 0; r < kWave; r += 16) {
        int32_t x[2] = {__builtin_amdgcn_readlane(w[0], r), __builtin_amdgcn_readlane(w[1], r)};
        T u;
        __builtin_memcpy(&u, x, 8);
        m = r == 0 ? u : (u < m ? u : m);
    }
    return m;
}

// Returns false if the list of running transfers would need more than `entries` entries: nothing of the configuration is
// final then, and run_bi_block does it from the start.
// K words of every set per thread, kWaves wavefronts (1 or kBlockWaves).
template <typename T, bool kSched, int K, int kWaves>
__device__ bool run_bi_wide(const Config<T> &c, int4 *red, uint64_t *rows, uint64_t *sets, int entries, const SchedOut &sched,
                            int64_t out_base, T *result, int32_t *status)
{
    constexpr int kThreads = kWaves * kWave;
    const int tid = static_cast<int>(threadIdx.x), lane = lane_id();
    const int wave = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = c.p, q = c.q;
    const int W = (p + 63) >> 6, kw = (W + kThreads - 1) / kThreads, w0 = tid * kw;
    const uint64_t root = tid == 0 ? UINT64_C(1) : 0;                      // processor 0: bit 0 of word 0
    const bool ragged = c.sz_last != c.sz, guardL = ragged && c.g_last > 0;
    const T kInf = CostTraits<T>::inf();

    uint64_t valid[K], sfree[K], rfree[K], compF[K], compL[K], lateL[K], rowNext[K];
    bool own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int w = w0 + k;
        own[k] = k < kw && w < W;
        valid[k] = !own[k] ? 0 : ((w == W - 1 && (p & 63)) ? (UINT64_C(1) << (p & 63)) - 1 : ~UINT64_C(0));
        rowNext[k] = 0;
    }
    // ---- the list: lane e of every wavefront holds entry e
    T se = 0, re = 0;
    bool mine = false, mineShort = false;
    uint64_t active = 0;                                 // ballot of `mine`
    const uint64_t full = entries >= kWave ? ~UINT64_C(0) : (UINT64_C(1) << entries) - 1;

    T t = 0, Tmax = 0;
    int ndone = 0, segStart = 0, jhi = -1, preJ = -1, turn = 0;
    int64_t emitted = 0;
    bool anySender = true;
    const int64_t max_events = 4 * static_cast<int64_t>(p) * q + 16;
    auto fetch = [&](int j) {                            // row j: who has sent segment j; rows nobody has visited are not written
        preJ = j;
#pragma unroll
        for (int k = 0; k < K; ++k) rowNext[k] = (j <= jhi && own[k]) ? rows[static_cast<size_t>(j) * W + w0 + k] : 0;
    };
    auto partial = [&](int a, int b, int d) -> const int4 * {
        int4 *const part = red + (turn & 1) * kBlockWaves;
        ++turn;
        if (lane == kWave - 1) part[wave] = make_int4(a, b, 0, d);
        __syncthreads();
        return part;
    };

    for (int64_t ev = 0;; ++ev) {
        // ---------------------------------------------------------------- advance time (Algorithm 2: t <- next port release)
        if (ev > max_events) { *status = PRS_CFG_STALLED; return true; }
        bool lateOnly = false;
        if (ev > 0) {
            // ends of sends and combines after t; and the instants at which the sender of a full segment may take in the
            // smaller last one, at which only the last segment is visited and which count only while a processor has a
            // free send port (nothing pairs otherwise before a port frees)
            T port = kInf, late = kInf;
            if (mine) {
                if (se > t) port = se;
                if (re > t && re < port) port = re;
                if (guardL && !mineShort && se > t + c.c_last) { const T v = se - c.c_last; if (v > t) late = v; }
            }
            T tn = wave_min_dpp<T>(port);
            if (guardL) {
                const T tl = wave_min_dpp<T>(late);
                lateOnly = anySender && tl < tn;
                if (lateOnly) tn = tl;
            }
            if (!(tn < kInf)) { *status = PRS_CFG_STALLED; return true; }
            t = tn;
        }
        int j = lateOnly ? q - 1 : segStart;
        fetch(j);
        // ---- port and computation sets from the transfers that still run
        {
            mine = mine && (se > t || re > t);
            active = ballot64(mine);
            const bool busy = se <= t && t < re, pend = t < se;            // receivers compute / will from se on
            // A transfer begun now must not run into that computation.  The entry began before t: against a segment of
            // its own size that settles it; against the other size the rounded sums are compared.
            const uint64_t sb = ballot64(mine && se > t), rb = ballot64(mine && re > t);
            const uint64_t cF = ballot64(mine && (busy || (pend && (!mineShort || t + c.c_full > se))));
            const uint64_t cL = ballot64(mine && (busy || (pend && (mineShort || !ragged || t + c.c_last > se))));
            // the combine of the smaller last segment, received now, would begin while this processor is still sending
            const uint64_t lt = ballot64(mine && guardL && !mineShort && se > t + c.c_last);
#pragma unroll
            for (int k = 0; k < K; ++k) { sfree[k] = rfree[k] = valid[k]; compF[k] = compL[k] = lateL[k] = 0; }
            sfree[0] &= ~root;                                             // the root never sends
            uint64_t left = active;
            while (left != 0) {                                            // four entries at a time: their loads are independent
                int e[4];
                uint64_t sm[4][K], rm[4][K];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    e[u] = left != 0 ? __builtin_ctzll(left) : e[u > 0 ? u - 1 : 0];
                    left &= left - 1;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const size_t at = static_cast<size_t>(e[u]) * 2 * W + w0 + k;
                        sm[u][k] = own[k] ? sets[at] : 0;
                        rm[u][k] = own[k] ? sets[at + W] : 0;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t ms = 0 - ((sb >> e[u]) & 1), mr = 0 - ((rb >> e[u]) & 1), mF = 0 - ((cF >> e[u]) & 1),
                                   mL = 0 - ((cL >> e[u]) & 1), mt = 0 - ((lt >> e[u]) & 1);
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        sfree[k] &= ~(sm[u][k] & ms); rfree[k] &= ~(rm[u][k] & mr);
                        compF[k] |= rm[u][k] & mF; compL[k] |= rm[u][k] & mL; lateL[k] |= sm[u][k] & mt;
                    }
                }
            }
        }
        // ---------------------------------------------------------------- visits (t, j)
        for (;;) {
            const bool past = j >= q;
            if (past && !guardL) break;                                    // only the late instants ask for free senders
            const bool last = j >= q - 1;
            if (preJ != j && !past) fetch(j);
            uint64_t row[K], fr[K], so[K], ro[K];
            int pf = 0, pm = 0, pso = 0, pro = 0, pu = 0;
            bool as = false, ar = false, any = false, cand = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                row[k] = rowNext[k];
                const uint64_t comp = last ? compL[k] : compF[k];
                const uint64_t s = sfree[k] & ~comp, r = rfree[k] & ~comp & ~(last ? lateL[k] : UINT64_C(0));
                const uint64_t memb = ~row[k] & valid[k];                  // still hold segment j (root: until done)
                const uint64_t sOK = memb & s, rOK = memb & r;
                fr[k] = sOK & rOK; so[k] = sOK ^ fr[k]; ro[k] = rOK ^ fr[k];
                pf += __popcll(fr[k]); pm += __popcll(memb); pso += __popcll(so[k]); pro += __popcll(ro[k]);
                pu += __popcll(s | r);
                as = as | (s != 0); ar = ar | (r != 0); any = any | (sfree[k] != 0);
                cand = cand | (((sfree[k] | rfree[k]) & ~comp & row[k]) != 0);
            }
            const int scanF = dpp_inclusive_scan(pf | (pm << 16)), sumO = dpp_inclusive_scan(pso | (pro << 16));
            const uint64_t some = ballot64(pu != 0);
            const int two = ballot64(pu > 1) != 0 ? 2 : (some == 0 ? 0 : ((some & (some - 1)) != 0 ? 2 : 1));
            const int mine4 = (ballot64(as) != 0 ? 1 : 0) | (ballot64(ar) != 0 ? 16 : 0) | (ballot64(any) != 0 ? 256 : 0) |
                              (ballot64(cand) != 0 ? 4096 : 0) | (two << 16);
            int4 theirs;
            if (kWaves > 1) {
                const int4 *const part = partial(scanF, sumO, mine4);
                theirs = part[lane & (kWaves - 1)];                        // lane w of eight has wavefront w's sums
            } else {
                theirs = make_int4(__builtin_amdgcn_readlane(scanF, kWave - 1), __builtin_amdgcn_readlane(sumO, kWave - 1), 0, mine4);
            }
            if (!past && j + 1 < q) fetch(j + 1);                          // on its way while this visit goes on
            auto total = [&](int v) { return kWaves > 1 ? __builtin_amdgcn_readfirstlane(dpp_sum8(v)) : v; };
            const int flags = total(theirs.w), either = flags >> 16;
            const int nf_ = total(theirs.x & 0xFFFF), remj = total(static_cast<int>(static_cast<uint32_t>(theirs.x) >> 16)) - 1;
            const int ns_ = total(theirs.y & 0xFFFF), nr_ = total(static_cast<int>(static_cast<uint32_t>(theirs.y) >> 16));
            anySender = (flags & 0xF00) != 0;
            if (past) break;
            // a pair needs a free send port and a free receive port on two different processors: without them only the last
            // segment, whose shorter transfer is kept out by fewer pending computations, is left to try
            if ((flags & 0xF) == 0 || (flags & 0xF0) == 0 || either < 2) {
                if (last) break;
                j = q - 1;
                continue;
            }
            if (remj == 0) {                                               // everybody has sent segment j
                if (j == segStart) ++segStart;
                ++j;
                continue;
            }
            int toSendLast, toRecvFirst;                                   // free processors go to the shorter list
            if (ns_ == nr_) {
                toSendLast = toRecvFirst = nf_ / 2;
            } else if (ns_ < nr_) {
                const int y = nr_ - ns_, mm = nf_ < y ? nf_ : y, xx = (nf_ - mm) / 2;
                toSendLast = mm + xx; toRecvFirst = xx;
            } else {
                const int y = ns_ - nr_, mm = nf_ < y ? nf_ : y, xx = (nf_ - mm) / 2;
                toRecvFirst = mm + xx; toSendLast = xx;
            }
            const int sN = ns_ + toSendLast, rN = nr_ + toRecvFirst;
            const int l = sN < rN ? sN : rN;
            const int at = j;
            if (j > jhi) {
                // a jump to the last segment can pass segments nobody has visited: their rows are empty
                for (int jj = jhi + 1; jj <= j; ++jj)
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (own[k]) rows[static_cast<size_t>(jj) * W + w0 + k] = 0;
                jhi = j;
            }
            ++j;
            if (l == 0) {
                // nobody paired although no candidate had already sent the segment: the candidates of later segments are a
                // subset of these, so only the last one can still pair at this t
                if ((flags & 0xF000) == 0) {
                    if (last) break;
                    j = q - 1;
                }
                continue;
            }
            // First l entries of each list.  Either the free processors even the lists out: the first of them receive, the last
            // send, an odd one in between does neither.  Or there are too few of them: all join the shorter list, and the longer
            // one, which has none, is cut.  So one search for a place is enough, and the places before my words are known
            // without another sum over the block.
            int exF = (scanF & 0xFFFF) - pf, exS = (sumO & 0xFFFF) - pso, exR = static_cast<int>(static_cast<uint32_t>(sumO) >> 16) - pro;
            if (kWaves > 1) {
                const bool before = (lane & (kWaves - 1)) < wave;
                exF += dpp_sum8(before ? theirs.x & 0xFFFF : 0); exS += dpp_sum8(before ? theirs.y & 0xFFFF : 0);
                exR += dpp_sum8(before ? static_cast<int>(static_cast<uint32_t>(theirs.y) >> 16) : 0);
            }
            uint64_t sset[K], rset[K];
            const bool cutS = sN > l, cutR = rN > l;
            const int odd = nf_ - toSendLast - toRecvFirst;
            const int posS = exS + (exF > nf_ - toSendLast ? exF - (nf_ - toSendLast) : 0), posR = exR + (exF < toRecvFirst ? exF : toRecvFirst);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int n = __popcll(fr[k]);
                const uint64_t firsts = lowest_bits_of_few(cutS ? so[k] : (cutR ? ro[k] : fr[k]), cutS ? l - exS : (cutR ? l - exR : toRecvFirst - exF), lane);
                uint64_t rest = fr[k] & ~firsts;
                if (odd != 0 && exF <= toRecvFirst && toRecvFirst < exF + n) rest &= rest - 1;
                sset[k] = cutS ? firsts : so[k] | (cutR ? fr[k] : rest);
                rset[k] = cutR ? firsts : ro[k] | (cutS ? fr[k] : firsts);
                exF += n; exS += __popcll(so[k]); exR += __popcll(ro[k]);
            }
            const T cj = last ? c.c_last : c.c_full, gj = last ? c.g_last : c.g_full;
            const T tc = t + cj, tr = tc + gj;
            if (!(tc > t)) { *status = PRS_CFG_STALLED; return true; }
            if ((active & full) == full) return false;
            if (kSched) {                                                  // e-th sender pairs with e-th receiver
                const int64_t o = out_base + emitted;
                for (int e = tid; e < l; e += kThreads) {
                    if (sched.seg) sched.seg[o + e] = at;
                    if (sched.tstart) static_cast<T *>(sched.tstart)[o + e] = t;
                }
                int32_t *src = sched.src ? sched.src + (o + posS) : nullptr, *dst = sched.dst ? sched.dst + (o + posR) : nullptr;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int base = (w0 + k) * 64;
                    if (src) {
                        src += emit_set_bits(src, static_cast<uint32_t>(sset[k]), base);
                        src += emit_set_bits(src, static_cast<uint32_t>(sset[k] >> 32), base + 32);
                    }
                    if (dst) {
                        dst += emit_set_bits(dst, static_cast<uint32_t>(rset[k]), base);
                        dst += emit_set_bits(dst, static_cast<uint32_t>(rset[k] >> 32), base + 32);
                    }
                }
            }
            emitted += l;
            const int e = __builtin_ctzll(~active);
            if (lane == e) { se = tc; re = tr; mine = true; mineShort = last && ragged; }
            active |= UINT64_C(1) << e;
            const bool late = guardL && !last && tc > t + c.c_last;         // these senders cannot take the last segment in yet
#pragma unroll
            for (int k = 0; k < K; ++k) {
                sfree[k] &= ~sset[k]; rfree[k] &= ~rset[k];
                if (late) lateL[k] |= sset[k];
                if (own[k]) {
                    sets[static_cast<size_t>(e) * 2 * W + w0 + k] = sset[k];
                    sets[static_cast<size_t>(e) * 2 * W + W + w0 + k] = rset[k];
                    rows[static_cast<size_t>(at) * W + w0 + k] = row[k] | sset[k];
                }
            }
            if (remj == l) {                                               // only the root is left: done after the last arrival
                if (tr > Tmax) Tmax = tr;
                if (++ndone == q) { *result = Tmax; return true; }
            }
        }
    }
}

template <typename T, bool kSched, int K>
__global__ __launch_bounds__(kBlockThreads) void bi_block_kernel(ConfigArrays cfg, int32_t p_max, int32_t q_max, int model,
                                                                 TimesOut times, SchedOut sched, PlanHeader *plan,
                                                                 const int32_t *order, int cls, int entries, int32_t state_p,
                                                                 int32_t state_q, char *slots, size_t slot_bytes)
{
    PRS_DYNAMIC_LDS(lds_raw);
    __shared__ long long s_ticket;
    __shared__ int s_done;
    const int tid = static_cast<int>(threadIdx.x);
    char *slot = slots + static_cast<size_t>(blockIdx.x) * slot_bytes;
    const BlockSlot sl = bi_block_slot(state_p, state_q);
    const int Wc = (state_p + 63) >> 6;
    int4 *red = reinterpret_cast<int4 *>(lds_raw + bb_align(static_cast<size_t>(Wc) * 8 * 7) + bb_align(static_cast<size_t>(Wc) * 2 * 2) + 512);
    const int32_t count = plan->class_count[cls], begin = plan->class_begin[cls];
    for (;;) {
        __syncthreads();
        if (tid == 0) s_ticket = static_cast<long long>(atomicAdd(&plan->ticket[cls], 1ULL));
        __syncthreads();
        const int64_t ticket = s_ticket;
        if (ticket >= count) break;
        const int64_t i = order[begin + ticket];
        Config<T> c = decode_config<T>(cfg, i, p_max, q_max);
        int32_t status = c.status;
        int64_t base = 0;
        if (kSched && status == PRS_CFG_OK) {
            base = sched.pair_offset[i];
            const int64_t cnt = static_cast<int64_t>(c.p - 1) * c.q;
            if (base < 0 || base + cnt > sched.pair_capacity) status = PRS_CFG_TOO_LARGE;
        }
        T result = CostTraits<T>::bad();
        if (status == PRS_CFG_OK) {
            bool done = false;
            uint64_t *const rows = reinterpret_cast<uint64_t *>(slot + sl.sent), *const sets = reinterpret_cast<uint64_t *>(slot + sl.sets);
            const int per_lane = (c.p + kWave * 64 - 1) / (kWave * 64);    // words of a set per lane of one wavefront
            if (per_lane <= (kSched ? kAloneWordsSched : kAloneWords)) {
                if (tid < kWave) {
                    if (kSched || per_lane <= 1) done = run_bi_wide<T, kSched, 1, 1>(c, red, rows, sets, entries, sched, base, &result, &status);
                    else if (per_lane <= 2) done = run_bi_wide<T, kSched, 2, 1>(c, red, rows, sets, entries, sched, base, &result, &status);
                    else done = run_bi_wide<T, kSched, kAloneWords, 1>(c, red, rows, sets, entries, sched, base, &result, &status);
                    if (tid == 0) s_done = done ? 1 : 0;
                }
                __syncthreads();
                done = s_done != 0;
            } else if (c.p <= kBlockThreads * 64) {
                done = run_bi_wide<T, kSched, 1, kBlockWaves>(c, red, rows, sets, entries, sched, base, &result, &status);
            } else if (c.p <= kBlockThreads * K * 64) {                    // always, where this kernel is launched
                done = run_bi_wide<T, kSched, K, kBlockWaves>(c, red, rows, sets, entries, sched, base, &result, &status);
            }
            if (!done) {
                __syncthreads();
                result = run_bi_block<T, kSched>(c, lds_raw, slot, sl, Wc, sched, base, &status);
            }
        }
        __syncthreads();
        if (tid == 0) {
            if (!kSched) write_closed_forms<T>(times, i, c, model);
            T *tg = static_cast<T *>(kSched ? sched.T_greedy : times.greedy);
            int32_t *cs = kSched ? sched.cfg_status : times.cfg_status;
            if (tg) tg[i] = status == PRS_CFG_OK ? result : CostTraits<T>::bad();
            if (cs) cs[i] = status;
        }
    }
}

template <typename T, bool kSched, int K>
static hipError_t launch_bi_block_as(const BiLaunch &L)
{
    hipLaunchKernelGGL((bi_block_kernel<T, kSched, K>), dim3(L.grid), dim3(kBlockThreads), L.lds_bytes, L.stream, L.cfg, L.p_max,
                       L.q_max, L.model, L.times, L.sched, L.plan, L.order, L.cls, L.list_entries, L.slot_p, L.slot_q, L.slots, L.slot_bytes);
    return hipGetLastError();
}
template <typename T, bool kSched>
static hipError_t launch_bi_block_t(const BiLaunch &L)
{
    if (L.p_max > kBlockThreads * 3 * 64) return hipErrorInvalidValue;     // no batch of this kernel
    return L.p_max > kWideProcs ? launch_bi_block_as<T, kSched, 3>(L) : launch_bi_block_as<T, kSched, kWideWords>(L);
}

hipError_t launch_bi_block(const BiLaunch &L)
{
    if (L.cost == PRS_COST_I64) return L.want_schedule ? launch_bi_block_t<int64_t, true>(L) : launch_bi_block_t<int64_t, false>(L);
    return L.want_schedule ? launch_bi_block_t<double, true>(L) : launch_bi_block_t<double, false>(L);
}

}  // namespace prs
