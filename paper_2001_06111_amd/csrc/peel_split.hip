// peel_split.hip - the peel of larger graphs: split into ranges of bitruss
// numbers by grid-wide sweeps, then finish each range by itself.
//
// Peeling level by level, as Algorithm 5 does, is a chain of tens of
// thousands of dependent rounds (75,000 for a 5M-edge power-law graph), and
// every round touches blooms across the graph.  The two-phase peeling of
// Lakhotia, Kannan and Prasanna (parallel peeling of bipartite networks)
// breaks the chain:
//   1. A sweep works at coarse levels.  It takes every remaining edge with
//      support at most hi, cascades to the fixpoint as the level-by-level
//      peel does, and calls the edges removed a part: their bitruss numbers
//      lie between the smallest support when the part began and hi.  A few
//      hundred rounds remove everything, and the survivors of a bloom take
//      one decrement per round for all of a round's kills, so there are
//      fewer decrements as well.
//   2. Within a part, edges are peeled level by level against the edges of
//      this and later parts only, which needs the wedges whose first-removed
//      edge lies in the part (regroup.hip).  Parts do not wait for each
//      other.  A part below kLeafEdges edges is peeled by one workgroup
//      (peel_leaf.hip); a larger one is a job of the next sweep, which
//      splits all such jobs at once, each at its own levels; a part of a
//      single level is done.
// The bitruss numbers are those of Algorithm 5: the edges of later parts
// outlive a part's levels, so they keep their wedges in its blooms.
//
// One sweep is one cooperative kernel.  All jobs advance in each round, each
// job through: select (a workgroup reads a sample of the job's remaining
// supports and sets hi so that about a target share of the edges and of the
// summed support lies below it), gather (the edges at or below hi become the
// frontier), rounds until no edge falls to hi.
//
// Whole calls, level by level (by the kernel that did only that) and split:
// 5M-edge Chung-Lu graph (75,000 rounds, bound by the 9 us a round's two grid
// barriers and chains take) 1.115 s and 0.239 s; 200k-edge graph 66.4 and 17.5
// ms; 400k-edge hub graph by BiT-PC 436 and 98 ms; 192 pool graphs in one batch
// 620 and 143 ms.
// The 5M graph's first sweep is now bound by memory-side requests (about
// 2e10/s of support atomics and random reads), a small graph's by the 10 to
// 15 us of a round.  The level-by-level form (the same kernel, its parts single
// levels) stays for graphs of few levels (few_levels below) and for callers
// whose memory does not hold the second copy of the index that the split
// needs (5M-edge graph 1.23 s, 250k 88 ms, 2M-edge request graph 2.17 s; the
// kernel that did only that took 1.10 s, 80 ms and 1.92 s).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <memory>

#include "peel_split.h"

namespace bt {

namespace {

enum : int32_t { kJobActive = 0, kJobDone = 1 };
constexpr int kGatherPerLane = 8;  // edges per lane of a gather item
constexpr uint32_t kGatherChunk = kWave * kGatherPerLane;
// Sweeps of at least this many edges run on every CU by default: they are
// bound by atomic throughput more than by the latency of their rounds (three of
// four CUs and all: 20M-edge hub graph 2.99 and 2.91 s, 17M-edge Chung-Lu graph
// 900 and 886 ms, 12M 635 and 623, 5M 229 and 229).  Below, the CUs left over
// peel leaves beside the sweep, and lighter peels of others.
constexpr int64_t kAllCusEdges = int64_t(1) << 24;
constexpr int32_t kLevelMax = INT_MAX - 1;  // above every support

struct alignas(128) JobState {
    int32_t state;
    int32_t level;      // hi of the current part
    int32_t part;
    int32_t n_parts;    // parts begun
    int32_t gmin[2];    // smallest remaining support above the level, by round parity
    int32_t fr[2];      // frontier items exist for the round of this parity
    int32_t e0, e1;
    int64_t gather_round, select_round;  // last scheduled (-1: none)
    int64_t target_n, target_w;          // edges and summed support a part should take
    float scale;        // of the targets: cascades add to what a part takes
    float est_n;        // edges the last select expected to take
    float rem_n;        // edges it saw remaining
    int32_t narrow;     // split by levels, not by edges (a job that came back whole)
    int32_t hi_bound;   // its bitruss numbers are at most this
    // Level by level: the list of the remaining edges below a threshold, which
    // gathers at levels below it scan.
    int32_t thresh;     // -1: none yet
    int32_t delta;      // how far the next threshold lies above its level
    int32_t listed;     // the last gather scanned the list
    uint32_t n_list;    // its entries
};

// Level by level, a gather that scanned all that remains at each of a graph's
// thousands of levels would take as long as the rounds in between (5M-edge
// graph: 10,500 levels, 40 us a gather).  A gather at or above the threshold
// scans the job's edges, sets a new threshold and lists the edges below it;
// later ones scan the list, to which decrements add the edges that they take
// below the threshold (5M-edge graph 1.44 -> 1.27 s, 2M-edge request graph 2.71
// -> 2.22 s).  Thresholds are moved so that a list holds some kListTarget edges
// in all (2^13, 2^15, 2^17 and 2^19: 1.30, 1.27, 1.27 and 1.30 s).  Ranges below
// kListLeast are scanned as they are (250,000 edges 94 ms, with lists 97), and
// those of graphs of few levels, whose edges would join a list in masses (1.5M
// uniform edges 22.5 ms, with lists 45).
constexpr uint32_t kListLeast = 1u << 18, kListTarget = 1u << 15;

// What a sweep kernel is made for.  A form each, as all together keep more
// values than the 128 registers that 16 waves have (level by level, 5M edges
// 1.55 -> 1.46 s; split 242 -> 240 ms).
enum SweepForm : int {
    kSplit,  // parts
    kMany,   // level by level, many jobs
    kOne,    // level by level, one job: its level is known without a load
};

// A piece of at most 64 wedges of a touched bloom; b < 0: none.
struct alignas(8) SweepBloomItem {
    int32_t b;
    uint32_t lo;  // its first wedge
};

struct SweepGatherItem {
    int32_t part;
    int32_t how;      // kGatherList, kGatherPack
    uint32_t lo, hi;  // edges, or places of P.list
};
constexpr int32_t kGatherList = 1;  // scans places of P.list
constexpr int32_t kGatherPack = 2;  // lists the edges below the threshold

struct SweepCtl {
    Counter nf[2], ntc[2], ngth[2], nsel[2];
    Counter updates, bloom_visits, touched, unbatched;
    Counter left;      // jobs not done
    Counter n_parts;   // parts begun
    u64 rounds;        // rounds run so far (a resumed launch starts at this round)
    u64 round_b;       // two-kernel rounds: the round of phase B
    u64 prof[4];       // BT_PEEL_PROFILE=1: block-0 clock ticks (decide, A, bar, B with bar)
    u64 yield_src;     // address of the host-written yield word (0: none)
    int32_t yielded;    // set when the launch ended early to give way
    int32_t pad;
};

// A wave reads the host's yield word every kYieldEvery rounds, and after
// kYieldTicks of the 100 MHz clock (50 us): the first rounds of a large graph's
// sweep take up to milliseconds each.
constexpr int64_t kYieldEvery = 16;
constexpr u64 kYieldTicks = 5000;
// In the count of the next round's selects, which every block reads between
// two rounds anyway: all of them end the launch there.  It may be set while the
// count still grows.
constexpr u64 kYieldBit = u64(1) << 63;

// Parts a job may begin in one sweep; the last takes everything left.
constexpr int32_t kMaxParts = 64;
constexpr int kSelBins = 256;     // floating bins: 3 mantissa bits
constexpr int64_t kSelSamples = 4096;  // edges a select looks at

// What the sweep keeps of a bloom: a kill reads it with the atomic that
// counts in it.
struct alignas(8) BloomRec {
    u64 kc;           // (live wedges at the round's start << 32) | kills of this round
    uint32_t w0, w1;  // its wedges
    int32_t part;     // the last part that touched it (level by level: the last job)
    int32_t done;     // chunks of it that phase B has finished
};

struct SweepArgs {
    SweepCtl *ctl;
    JobState *js;
    int32_t n_jobs;
    SplitPart *parts;
    int32_t *sup;
    EdgeMark *mark;
    uint8_t *dead;      // per wedge
    BloomRec *bloom;
    int32_t *wedge_k;
    const int32_t *wea, *web;
    const int64_t *link_off;
    const uint3 *link;
    uint32_t n_w;
    int32_t *list;      // level by level: the jobs' lists, each where its edges are
    int32_t short_a, short_b;  // items that fill a wave in phases A, B; 0: most are long
    uint32_t reserve;   // slots that a wave may leave over in a phase
    FrontItem *front[2];  // {edge, part, links [lo, hi)}
    SweepBloomItem *tc[2];
    SweepGatherItem *gth[2];
    int32_t *sel[2];
};

__device__ __forceinline__ uint32_t chunks_of(uint32_t lo, uint32_t hi) {
    return (hi - lo + kLinkChunk - 1) / kLinkChunk;
}

__device__ __forceinline__ void set_front_flag(const SweepArgs &P, int32_t job, int q) {
    st(&P.js[job].fr[q], 1);
}

// The same for the jobs of the lanes with `on`; `last` is the job (uniform over
// the wave) whose flag the wave set last in this phase.  Stores to one
// address queue at the memory side, so a wave sets a job's flag once (a
// uniform graph of 4M edges, whose every step takes edges: 152 -> 93 ms).
// All 64 lanes call.
template <SweepForm F>
__device__ __forceinline__ void set_front_flags(const SweepArgs &P, bool on, int32_t part, int q,
                                                int32_t &last) {
    const int32_t job = !on ? -1 : F != kSplit ? part : ld(&P.parts[part].job);
    unsigned long long who = __ballot(on && job != last);
    while (who) {
        last = __shfl(job, __ffsll(who) - 1, kWave);
        if (lane_id() == 0) set_front_flag(P, last, q);
        who &= ~__ballot(job == last);
    }
}

// A wave's reservation of a work list's slots.  All waves of a round append
// to two lists, and one counter takes an atomic every few nanoseconds: with an
// atomic per step of a wave those counters bounded large rounds (33 ms of a
// 5M-edge graph's first sweep in phase A).  In a round of several items a
// wave, a wave therefore reserves twice its items' number of slots at a time
// (up to kReserve) and fills what it leaves over with null items, at most half
// as many as the round had.
constexpr uint32_t kReserve = 128;
// Slots that the waves of a phase may leave over in all.  Their lists take 80
// bytes a slot, 30 MB at kReserve a wave, which a caller short of memory has
// not counted on for a small graph: at most 64 bytes an edge there.
int64_t spare_slots(int64_t m, int64_t waves, bool least) {
    const int64_t all = waves * kReserve;
    return least ? std::min(all, m * 4 / 5) : all;
}
struct Reserve {
    uint32_t base = 0, left = 0;  // lists hold fewer than 2^32 items
};
// Slots of a step's items 0, 1, ...: the rest of the reservation, then a new one.
struct Slots {
    uint32_t old_base, new_base, old_left;
    __device__ uint32_t operator()(uint32_t i) const {
        return i < old_left ? old_base + i : new_base + (i - old_left);
    }
};

// Slots for n0 items of one list and n1 of another (uniform over the wave);
// both counters' atomics are issued together.  With grow 0 nothing is left over.
__device__ __forceinline__ void reserve2(Reserve &R0, uint32_t n0, u64 *k0, Reserve &R1,
                                         uint32_t n1, u64 *k1, uint32_t grow, Slots &S0,
                                         Slots &S1) {
    const uint32_t x0 = n0 > R0.left ? n0 - R0.left : 0u, x1 = n1 > R1.left ? n1 - R1.left : 0u;
    const uint32_t a0 = x0 ? max(x0, grow) : 0u, a1 = x1 ? max(x1, grow) : 0u;
    int r = 0;
    if (a0 | a1) {
        const uint32_t a = lane_id() == 0 ? a0 : a1;
        if (lane_id() < 2 && a) r = (int)(uint32_t)atomicAdd(lane_id() == 0 ? k0 : k1, (u64)a);
    }
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane(r, 0);
    const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane(r, 1);
    S0 = Slots{R0.base, r0, R0.left};
    S1 = Slots{R1.base, r1, R1.left};
    if (x0) {
        R0.base = r0 + x0;
        R0.left = a0 - x0;
    } else {
        R0.base += n0;
        R0.left -= n0;
    }
    if (x1) {
        R1.base = r1 + x1;
        R1.left = a1 - x1;
    } else {
        R1.base += n1;
        R1.left -= n1;
    }
}

// Each lane's cnt pieces of bloom b, whose wedges begin at lo, as items at slots
// S(at), ...: a lane writes its first, the whole wave the others of a longer
// range.  All 64 lanes call.
__device__ __forceinline__ void put_blooms(SweepBloomItem *list, const Slots &S, uint32_t cnt,
                                           uint32_t at, int32_t b, uint32_t lo) {
    const auto put = [&](uint32_t slot, int32_t bloom, uint32_t w) {
        st(reinterpret_cast<u64 *>(&list[slot]), ((u64)w << 32) | (uint32_t)bloom);
    };
    if (cnt) put(S(at), b, lo);
    unsigned long long big = __ballot(cnt > 1);
    while (big) {
        const int l = __ffsll(big) - 1;
        big &= big - 1;
        const uint32_t n = __shfl(cnt, l, kWave), a = __shfl(at, l, kWave), w = __shfl(lo, l, kWave);
        const int32_t lb = __shfl(b, l, kWave);
        for (uint32_t c = 1 + lane_id(); c < n; c += kWave) put(S(a + c), lb, w + c * kWedgeChunk);
    }
}

// The same for the links of an edge that joins a part and goes at `round`
// (lanes with take); an edge without links needs no item.
template <SweepForm F>
__device__ __forceinline__ void put_fronts(const SweepArgs &P, FrontItem *list, const Slots &S,
                                           bool take, uint32_t cnt, uint32_t at, int32_t e,
                                           int32_t part, int32_t level, int32_t round,
                                           uint32_t lo, uint32_t hi) {
    if (take) st(&P.mark[e].v, edge_mark(F != kSplit ? level : part, round));
    if (cnt) st_item(&list[S(at)], FrontItem{e, part, lo, min(lo + (uint32_t)kWave, hi)});
    unsigned long long big = __ballot(cnt > 1);
    while (big) {
        const int l = __ffsll(big) - 1;
        big &= big - 1;
        const uint32_t n = __shfl(cnt, l, kWave), a = __shfl(at, l, kWave);
        const int32_t le = __shfl(e, l, kWave), lp = __shfl(part, l, kWave);
        const uint32_t llo = __shfl(lo, l, kWave), lhi = __shfl(hi, l, kWave);
        for (uint32_t c = 1 + lane_id(); c < n; c += kWave) {
            const uint32_t x = llo + c * kWave;
            st_item(&list[S(a + c)], FrontItem{le, lp, x, min(x + (uint32_t)kWave, lhi)});
        }
    }
}

// Null items in the slots a wave leaves over at the end of a phase: a bloom
// item of no bloom (taken as the dead wedge past the last one), a frontier
// item of no edge.
__device__ __forceinline__ void fill_blooms(SweepBloomItem *list, const Reserve &R) {
    for (uint32_t i = lane_id(); i < R.left; i += kWave)
        st(reinterpret_cast<u64 *>(&list[R.base + i]), (u64)0xffffffffu);
}
__device__ __forceinline__ void fill_fronts(FrontItem *list, const Reserve &R) {
    for (uint32_t i = lane_id(); i < R.left; i += kWave)
        st_item(&list[R.base + i], FrontItem{-1, 0, 0u, 1u});
}

// Gather items over edges (or places) [e0, e0 + n) for phase B of this round, of
// parity p; each lane with n > 0 has its own.  All 64 lanes call.
__device__ __forceinline__ void put_gather(const SweepArgs &P, int p, int32_t part, uint32_t e0,
                                           uint32_t n, int32_t how) {
    const uint32_t cnt = (n + kGatherChunk - 1) / kGatherChunk;
    u64 base[3];
    wave_alloc3(cnt, &P.ctl->ngth[p].v, 0u, nullptr, 0u, nullptr, base);
    unsigned long long who = __ballot(cnt != 0);
    while (who) {
        const int l = __ffsll(who) - 1;
        who &= who - 1;
        const uint32_t nc = __shfl(cnt, l, kWave), ln = __shfl(n, l, kWave);
        const u64 b = __shfl(base[0], l, kWave);
        const int32_t lp = __shfl(part, l, kWave);
        const uint32_t le = __shfl(e0, l, kWave);
        const int32_t lh = __shfl(how, l, kWave);
        for (uint32_t c = lane_id(); c < nc; c += kWave) {
            const uint32_t a = c * kGatherChunk;
            st_item(&P.gth[p][b + c], SweepGatherItem{lp, lh, le + a, le + min(a + kGatherChunk, ln)});
        }
    }
}

// What each of this thread's jobs does next, decided at the start of round r
// (parity p) from what the last round left: rounds while there is a
// frontier; after a gather that took nothing, a gather at the smallest
// support it saw; else a select for the next part.  A gather runs in phase B
// of this round, where nothing else touches its job: one in the next round's
// phase A cost each level and part a round more (level by level, 250,000 edges
// 8,145 -> 7,155 rounds, 105 -> 99 ms).
template <SweepForm F>
__device__ void sweep_decide(const SweepArgs &P, int64_t r, int p, int64_t tid, int64_t nthreads) {
    const int q = p ^ 1;
    for (int64_t g0 = tid - lane_id(); g0 < P.n_jobs; g0 += nthreads) {
        const int64_t g = g0 + lane_id();
        bool gather = false, select = false;
        uint32_t e0 = 0, n = 0;
        int32_t part = 0, how = 0;
        if (g < P.n_jobs) {
            JobState *J = &P.js[g];
            const int32_t state = ld(&J->state);
            const int64_t gr = ld(&J->gather_round), sr = ld(&J->select_round);
            const int32_t fr = ld(&J->fr[p]);
            const int32_t gm = ld(&J->gmin[q]);
            const int32_t level = ld(&J->level);
            part = ld(&J->part);
            e0 = (uint32_t)ld(&J->e0);
            n = (uint32_t)ld(&J->e1) - e0;
            if (state != kJobDone) {
                if (fr) st(&J->fr[p], 0);
                if (!fr && sr != r) {
                    int32_t next = INT_MAX;
                    if (gr == r - 1) {
                        next = gm;
                        // Nothing is left in the list.
                        if (F != kSplit && gm == INT_MAX && ld(&J->listed)) next = ld(&J->thresh);
                        if (next == INT_MAX) {  // nothing remains
                            st(&J->state, (int32_t)kJobDone);
                            atomicAdd(&P.ctl->left.v, ~0ull);
                        }
                    } else if (level >= kLevelMax) {
                        // the part took everything
                        st(&J->state, (int32_t)kJobDone);
                        atomicAdd(&P.ctl->left.v, ~0ull);
                    } else if (F != kSplit) {
                        next = level + 1;
                        atomicAdd(&J->n_parts, 1);
                    } else {
                        select = true;
                        st(&J->select_round, r + 1);
                    }
                    if (next != INT_MAX) {
                        gather = true;
                        st(&J->level, next);
                        st(&P.parts[part].hi, next);
                        st(&J->gather_round, r);
                        st(&J->gmin[p], (int32_t)INT_MAX);
                        if (F != kSplit) {
                            if (P.list && n >= kListLeast) {
                                const int32_t t = ld(&J->thresh);
                                const uint32_t held = ld(&J->n_list);
                                if (next < t) {
                                    how = kGatherList;
                                    n = held;
                                } else {
                                    how = kGatherPack;
                                    int32_t d = ld(&J->delta);
                                    if (t >= 0 && held > 2 * kListTarget) d /= 2;
                                    else if (t >= 0 && held < kListTarget) d = min(2 * d + 1, 1 << 29);
                                    const int32_t t1 =
                                        (int32_t)min((int64_t)next + 1 + d, (int64_t)INT_MAX);
                                    st(&J->delta, d);
                                    st(&J->thresh, t1);
                                    st(&J->n_list, 0u);
                                    st(&P.parts[part].lo, t1);
                                }
                            }
                            st(&J->listed, how & kGatherList);
                        }
                    }
                }
            }
        }
        if (!__any(gather || select)) continue;
        put_gather(P, p, part, e0, gather ? n : 0u, how);
        const u64 slot = wave_alloc(select ? 1u : 0u, &P.ctl->nsel[q].v) & ~kYieldBit;
        if (select) st(&P.sel[q][slot], (int32_t)g);
    }
}

// Floating bins of d >= 1 with three mantissa bits, and the smallest value
// past a bin.
__device__ __forceinline__ int sel_bin(uint32_t d) {
    const int l = 31 - __clz((int)d);
    return l <= 3 ? (int)d : (int)((l - 3) * 8 + (int)(d >> (l - 3)));
}
__device__ __forceinline__ int64_t sel_end(int b) {
    if (b < 16) return (int64_t)b + 1;
    const int sh = b / 8 - 1;
    return (int64_t)(b % 8 + 8 + 1) << sh;
}

// Begins a job's next part: from a sample of its remaining supports, the
// largest level below which no more than the targets lie (at least the
// smallest support sampled), and the gather at it in phase B of this round.  A job
// that came back whole from the last sweep (some range's cascade took all of
// it) is cut into sixteenths of its range of levels instead, down to single
// levels.  One workgroup; all its threads call.
__device__ void sweep_select(const SweepArgs &P, int32_t g, int64_t r, int p) {
    __shared__ uint32_t s_n[kSelBins];
    __shared__ int32_t s_mn, s_mx;
    JobState *J = &P.js[g];
    const int32_t e0 = ld(&J->e0), e1 = ld(&J->e1);
    const int64_t n = e1 - e0;
    const int64_t samples = n < kSelSamples ? n : kSelSamples;
    const u64 step = samples ? ((u64)n << 31) / (u64)samples : 0;  // 31-bit fraction
    for (int i = threadIdx.x; i < kSelBins; i += blockDim.x) s_n[i] = 0;
    if (threadIdx.x == 0) {
        s_mn = INT_MAX;
        s_mx = -1;
    }
    __syncthreads();
    // Four samples' supports at a time, INT_MAX where the edge is gone.
    const auto sample4 = [&](int64_t i0, int32_t (&v)[4]) {
        int32_t ph[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + (int64_t)k * blockDim.x;
            ph[k] = 0;
            v[k] = INT_MAX;
            if (i < samples) {
                const int64_t e = e0 + (int64_t)(((u64)i * step) >> 31);
                ph[k] = mark_part(ld(&P.mark[e].v));
                v[k] = ld(&P.sup[e]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = ph[k] < 0 ? v[k] : INT_MAX;
    };
    int32_t mn = INT_MAX, mx = -1;
    for (int64_t i = threadIdx.x; i < samples; i += 4 * (int64_t)blockDim.x) {
        int32_t v[4];
        sample4(i, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            mn = min(mn, v[k]);
            mx = max(mx, v[k] == INT_MAX ? -1 : v[k]);
        }
    }
    mn = wave_min(mn);
    mx = -wave_min(-mx);
    if (lane_id() == 0) {
        atomicMin(&s_mn, mn);
        atomicMax(&s_mx, mx);
    }
    __syncthreads();
    mn = s_mn;
    mx = s_mx;
    for (int64_t i = threadIdx.x; i < samples; i += 4 * (int64_t)blockDim.x) {
        int32_t v[4];
        sample4(i, v);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (v[k] != INT_MAX) atomicAdd(&s_n[sel_bin((uint32_t)(v[k] - mn) + 1u)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        // One wave: four bins a lane, their prefix sums, and the first bin
        // past a target.
        const int b0 = 4 * lane_id();
        uint32_t cn[4];
        float cw[4], lw = 0.f;  // summed support of a bin, from its middle
        uint32_t ln = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int b = b0 + k;
            cn[k] = s_n[b];
            cw[k] = cn[k] ? (float)cn[k] * ((float)mn + 0.5f * (float)(sel_end(b - 1) + sel_end(b)) - 1.f)
                          : 0.f;
            ln += cn[k];
            lw += cw[k];
        }
        const uint32_t in = wave_inclusive_sum<uint32_t>(ln);
        const float iw = wave_inclusive_sum<float>(lw);
        const float up = samples ? (float)n / (float)samples : 1.f;
        const float rem = (float)wave_last(in) * up;
        const float all = __shfl(iw, kWave - 1, kWave);
        const int32_t np = ld(&J->n_parts), level = ld(&J->level);
        const int64_t tn0 = ld(&J->target_n);
        int64_t tw = ld(&J->target_w);
        float scale = ld(&J->scale);
        if (np == 0) {  // the job's whole support, from the sample
            tw = (int64_t)(all * up * ((float)tn0 / (float)(n > 0 ? n : 1)));
        } else {
            // The last part took rem(then) - rem(now) edges; what it was
            // expected to take, over that, tells how far to aim below.
            const float took = ld(&J->rem_n) - rem, est = ld(&J->est_n);
            if (took > 0.f && est > 0.f)
                scale = fminf(1.f, fmaxf(0.05f, 0.5f * scale + 0.5f * est / took));
        }
        const float tn = (float)tn0 * scale, tws = (float)tw * scale;
        int cut = kSelBins;  // this lane's first bin past a target
        float an = (float)(in - ln) * up, aw = (iw - lw) * up;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float bn = (float)cn[k] * up, bw = cw[k] * up;
            if (cut == kSelBins && cn[k] && an > 0.f && (an + bn > tn || aw + bw > tws))
                cut = b0 + k;
            an += bn;
            aw += bw;
        }
        cut = wave_min(cut);
        int last = -1;  // the last bin taken
        uint32_t taken = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (b0 + k < cut && cn[k]) {
                last = b0 + k;
                taken += cn[k];
            }
        last = -wave_min(-last);
        taken = wave_sum(taken);
        if (lane_id() == 0) {
            int64_t end = (int64_t)kLevelMax + 1;  // of the supports taken
            if (np + 1 < kMaxParts && mn != INT_MAX) {
                if (ld(&J->narrow)) {
                    const int64_t top = min(ld(&J->hi_bound), mx);
                    const int64_t width = (top - mn + 1) / 16;
                    // Of single levels the gather finds the exact minimum: a
                    // part at the old level takes nothing and jumps to it.
                    end = width > 1 ? (int64_t)mn + width : (int64_t)level + 1;
                } else if (cut < kSelBins) {
                    end = (int64_t)mn + sel_end(last) - 1;
                }
            }
            const int32_t hi = (int32_t)(end - 1 < kLevelMax ? end - 1 : kLevelMax);
            const int32_t part = (int32_t)atomicAdd(&P.ctl->n_parts.v, 1ull);
            st(&P.parts[part].hi, hi);
            st(&P.parts[part].lo, (int32_t)INT_MAX);
            st(&P.parts[part].job, g);
            st(&P.parts[part].pad, 0);
            st(&J->target_w, tw);
            st(&J->scale, scale);
            st(&J->est_n, (float)taken * up);
            st(&J->rem_n, rem);
            st(&J->n_parts, np + 1);
            st(&J->level, hi);
            st(&J->part, part);
            st(&J->gather_round, r);
            st(&J->gmin[p], (int32_t)INT_MAX);
            s_mn = part;
        }
    }
    __syncthreads();
    if (threadIdx.x < kWave)  // one wave writes the gather's items
        put_gather(P, p, s_mn, (uint32_t)e0, threadIdx.x == 0 ? (uint32_t)n : 0u, 0);
    __syncthreads();
}

// The smallest support a wave's gather items saw; most waves find a smaller
// one there already.
__device__ __forceinline__ void flush_min(const SweepArgs &P, int p, int32_t job, int32_t mn) {
    if (lane_id() == 0 && mn != INT_MAX && mn < ld(&P.js[job].gmin[p]))
        atomicMin(&P.js[job].gmin[p], mn);
}

// A gather item: remaining edges at or below the part's level become the next
// frontier; the smallest support above it is kept for a jump, the smallest
// taken as the part's lower bound.  The smallest is kept by the wave until its
// items' job changes: one counter takes an atomic every few nanoseconds.
template <SweepForm F>
__device__ __forceinline__ void sweep_gather(const SweepArgs &P, int64_t r, int p,
                                             const SweepGatherItem it, int32_t &mn_job,
                                             int32_t &mn_all, int32_t &flagged) {
    SweepCtl *C = P.ctl;
    const int q = p ^ 1;
    const int32_t level = ld(&P.parts[it.part].hi), job = ld(&P.parts[it.part].job);
    int32_t ph[kGatherPerLane], sv[kGatherPerLane];
    uint32_t ed[kGatherPerLane];
#pragma unroll
    for (int k = 0; k < kGatherPerLane; ++k) {
        const uint32_t i = it.lo + k * kWave + lane_id();
        ed[k] = i;
        if (F != kSplit && (it.how & kGatherList) && i < it.hi) ed[k] = (uint32_t)ld(&P.list[i]);
    }
#pragma unroll
    for (int k = 0; k < kGatherPerLane; ++k) {
        const uint32_t e = ed[k];
        ph[k] = 0;
        sv[k] = INT_MAX;
        if (it.lo + k * kWave + lane_id() < it.hi) {
            ph[k] = mark_part(ld(&P.mark[e].v));
            sv[k] = ld(&P.sup[e]);
        }
    }
    int32_t mn = INT_MAX, lowest = INT_MAX;
    uint32_t take = 0;
#pragma unroll
    for (int k = 0; k < kGatherPerLane; ++k)
        if (ph[k] < 0) {
            if (sv[k] <= level) {
                take |= 1u << k;
                lowest = min(lowest, sv[k]);
            } else {
                mn = min(mn, sv[k]);
            }
        }
    if (__ballot(take != 0)) {
        uint32_t lo[kGatherPerLane], hi[kGatherPerLane], tot = 0;
#pragma unroll
        for (int k = 0; k < kGatherPerLane; ++k) {
            const uint32_t e = ed[k];
            lo[k] = hi[k] = 0;
            if ((take >> k) & 1u) {
                lo[k] = (uint32_t)P.link_off[e];
                hi[k] = (uint32_t)P.link_off[(int64_t)e + 1];
            }
            tot += chunks_of(lo[k], hi[k]);
        }
        u64 base[3];
        wave_alloc3(tot, &C->nf[q].v, 0u, nullptr, 0u, nullptr, base);
        const Slots S{0, 0, 0xffffffffu};
        uint32_t at = (uint32_t)base[0];
#pragma unroll
        for (int k = 0; k < kGatherPerLane; ++k) {
            const uint32_t cnt = chunks_of(lo[k], hi[k]);
            put_fronts<F>(P, P.front[q], S, (take >> k) & 1u, cnt, at,
                       (int32_t)ed[k], it.part, level, (int32_t)(r + 1), lo[k], hi[k]);
            at += cnt;
        }
        lowest = wave_min(lowest);
        if (lane_id() == 0) {
            if (job != flagged) set_front_flag(P, job, q);
            if (F == kSplit) atomicMin(&P.parts[it.part].lo, lowest);
        }
        flagged = job;
    }
    if (F != kSplit && (it.how & kGatherPack)) {
        const int32_t t = ld(&P.js[job].thresh);
        uint32_t keep = 0;
#pragma unroll
        for (int k = 0; k < kGatherPerLane; ++k)
            keep += ph[k] < 0 && sv[k] > level && sv[k] < t ? 1u : 0u;
        if (__ballot(keep != 0)) {
            const uint32_t inc = wave_inclusive_sum<uint32_t>(keep);
            uint32_t base = 0;
            if (lane_id() == 0) base = atomicAdd(&P.js[job].n_list, wave_last(inc));
            uint32_t at = (uint32_t)ld(&P.js[job].e0) +
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + inc - keep;
#pragma unroll
            for (int k = 0; k < kGatherPerLane; ++k)
                if (ph[k] < 0 && sv[k] > level && sv[k] < t) st(&P.list[at++], (int32_t)ed[k]);
        }
    }
    mn = wave_min(mn);
    if (job != mn_job) {
        flush_min(P, p, mn_job, mn_all);
        mn_job = job;
        mn_all = INT_MAX;
    }
    mn_all = min(mn_all, mn);
}


// Work items of a phase per wave and step: one while there are few items, so
// that a small round spreads over the chip; up to 64, one a lane, when there
// are more (most items hold a few links or wedges, which the wave then spreads
// over its lanes).  Items are few while a wave has fewer than four of them, as
// the longest bound the phase; where most are short (`least` > 0), a wave takes
// its share in one step and at least as many as fill its lanes, since each
// step also takes slots from counters that all waves share (a uniform graph of
// 117,248 edges, items of two to five: 89 -> 44 us a round).
__device__ __forceinline__ uint32_t items_per_step(u64 n, int64_t nwaves, int32_t least) {
    const u64 per = least > 0 ? max((n + (u64)nwaves - 1) / (u64)nwaves, (u64)least)
                              : n / (u64)(4 * nwaves);
    return per < 1 ? 1u : per > kWave ? (uint32_t)kWave : (uint32_t)per;
}

// Whether an edge's removal kills a link's wedge: the twin is still there, or
// goes in the same round and is the larger of the two.
__device__ __forceinline__ bool kills(bool has, int32_t e, int32_t twin, int32_t tround, int32_t now) {
    return has && e >= 0 && tround >= now && !(tround == now && twin < e);
}

// Level by level: edges that fell below their job's threshold (lanes with on)
// join its list.  All 64 lanes call.
__device__ __forceinline__ void list_edges(const SweepArgs &P, bool on, int32_t job, int32_t e) {
    unsigned long long who = __ballot(on);
    while (who) {
        const int l = __ffsll(who) - 1;
        const int32_t j = __shfl(job, l, kWave);
        const unsigned long long same = __ballot(on && job == j);
        uint32_t base = 0;
        if (lane_id() == l) base = atomicAdd(&P.js[j].n_list, (uint32_t)__popcll(same));
        base = (uint32_t)__shfl((int)base, l, kWave) + (uint32_t)ld(&P.js[j].e0);
        if ((same >> lane_id()) & 1)
            st(&P.list[base + (uint32_t)__popcll(same & lanemask_lt())], e);
        who &= ~same;
    }
}

// A part's level, and level by level its threshold (INT_MIN: no list).
template <SweepForm F>
__device__ __forceinline__ int2 part_level(const SweepArgs &P, int32_t part, int2 one) {
    if (F == kSplit) return make_int2(ld(&P.parts[part].hi), 0);
    if (F == kOne) return one;
    const u64 v = ld(reinterpret_cast<const u64 *>(&P.parts[part].hi));
    return make_int2((int32_t)(uint32_t)v, (int32_t)(v >> 32));
}

// Phase A of the only job of a level-by-level peel, with few items: one a wave
// and step.  Such a round is a chain of waits for memory, so what does not
// depend on each other is asked for together: the item; its links; all that a
// link may need (the twin's mark and links, the bloom's record); the kill and
// the twin's decrement; the slots (250,000 edges 94.5 -> 89 ms, 5M 1.27 -> 1.23 s).
// Where many items hide the waits that only costs requests (split, 192 pool
// graphs: 144 -> 148 ms).
__device__ __forceinline__ void sweep_phase_a_few(const SweepArgs &P, int64_t r, int p, u64 nf,
                                                  int2 one, int64_t wid, int64_t nwaves,
                                                  uint32_t &upd) {
    SweepCtl *C = P.ctl;
    const int q = p ^ 1;
    const int32_t now = (int32_t)r, level = one.x, thresh = one.y;
    bool flagged = false;
    FrontItem it{};
    if (wid < (int64_t)nf) it = ld_item(&P.front[p][wid]);
    for (int64_t i = wid; i < (int64_t)nf; i += nwaves) {
        const FrontItem cur = it;
        if (i + nwaves < (int64_t)nf) it = ld_item(&P.front[p][i + nwaves]);  // loaded early
        const int32_t e = cur.e;
        const uint32_t j = cur.lo + lane_id();
        const bool has = j < cur.hi;
        uint3 lk = make_uint3(0, 0, kFixedBit);
        if (has) lk = P.link[j];
        const bool tfix = (lk.z & kFixedBit) != 0;
        const int32_t twin = (int32_t)(lk.z & kEdgeMask);
        BloomRec *const B = &P.bloom[lk.y];
        int32_t tround = INT_MAX;
        u64 kc = 0;
        uint2 w01 = make_uint2(0, 0);
        uint32_t tlo = 0, thi = 0;
        if (has) {
            kc = ld(&B->kc);
            w01 = *reinterpret_cast<const uint2 *>(&B->w0);
            if (!tfix) {
                tround = mark_round(ld(&P.mark[twin].v));
                tlo = (uint32_t)P.link_off[twin];
                thi = (uint32_t)P.link_off[(int64_t)twin + 1];
            }
        }
        const bool kill = kills(has, e, twin, tround, now);
        const int32_t d = (int32_t)(kc >> 32) - 1;
        const bool dec = kill && d > 0 && !tfix && tround != now;
        u64 old = 1;
        int32_t otw = 0;
        if (kill) {  // both atomics issue before either result is used
            old = atomicAdd(&B->kc, (u64)1);
            if (dec) otw = atomicSub(&P.sup[twin], d);
            st(&P.dead[lk.x], (uint8_t)1);
        }
        const bool first = kill && d > 0 && (uint32_t)old == 0;
        const bool tf = dec && otw > level && otw - d <= level;
        if (__ballot(first || tf)) {
            const uint32_t nch = first ? (w01.y - w01.x + kWedgeChunk - 1) / kWedgeChunk : 0u;
            const uint32_t tk = tf ? chunks_of(tlo, thi) : 0u;
            u64 base[3];
            wave_alloc3(nch, &C->ntc[p].v, tk, &C->nf[q].v, 0u, nullptr, base);
            const Slots S{0, 0, 0xffffffffu};
            put_blooms(P.tc[p], S, nch, (uint32_t)base[0], (int32_t)lk.y, w01.x);
            put_fronts<kOne>(P, P.front[q], S, tf, tk, (uint32_t)base[1], twin, 0, level, now + 1,
                             tlo, thi);
            if (!flagged && __ballot(tf)) {
                if (lane_id() == 0) set_front_flag(P, 0, q);
                flagged = true;
            }
        }
        list_edges(P, dec && otw >= thresh && otw - d < thresh && otw - d > level, 0, twin);
        upd += dec ? 1 : 0;
    }
}

// Phase A: the frontier's wedges are killed; each kill counts in its bloom,
// and the twin edge loses all of its butterflies in the bloom.  A wedge is
// alive unless its twin was removed in an earlier round; where both edges are
// in the frontier the smaller one kills it.  (A wedge that outlived its bloom
// is killed for nothing: the bloom has no butterfly left to take.)  Bound by
// random accesses: a link reads its twin's mark; a kill adds two atomics and
// a byte, a bloom's first kill one read of its record.
template <SweepForm F>
__device__ __forceinline__ void sweep_phase_a(const SweepArgs &P, int64_t r, int p, u64 nf, int2 one,
                                              int64_t wid, int64_t nwaves, u64 *mask,
                                              uint32_t &upd) {
    SweepCtl *C = P.ctl;
    const int q = p ^ 1;
    const int32_t now = (int32_t)r;
    const uint32_t per = items_per_step(nf, nwaves, P.short_a);
    if (F == kOne && per == 1)
        return sweep_phase_a_few(P, r, p, nf, one, wid, nwaves, upd);
    const uint32_t grow = per > 1 ? min(2 * per, P.reserve) : 0u;
    Reserve rb, rf;
    int32_t flagged = -1;
    for (int64_t g0 = wid * per; g0 < (int64_t)nf; g0 += nwaves * per) {
        const bool ok = (uint32_t)lane_id() < per && g0 + lane_id() < (int64_t)nf;
        FrontItem it{0, 0, 0, 0};
        int2 level_l = make_int2(0, 0);
        if (ok) {
            it = ld_item(&P.front[p][g0 + lane_id()]);
            level_l = part_level<F>(P, it.part, one);
        }
        const uint32_t n = ok ? it.hi - it.lo : 0u;
        const uint32_t inc = wave_inclusive_sum<uint32_t>(n);
        const uint32_t start = inc - n;
        const uint32_t total = wave_last(inc);
        for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
            const int src = per == 1 ? 0 : item_of(ok, start, t0, mask);
            const uint32_t x = t0 + lane_id();
            const bool has = x < total;
            const uint32_t j = __shfl(it.lo - start, src, kWave) + x;
            const int32_t e = __shfl(it.e, src, kWave), part = __shfl(it.part, src, kWave);
            uint3 lk = make_uint3(0, 0, kFixedBit);
            int32_t tround = INT_MAX;
            if (has) {
                lk = P.link[j];
                if (!(lk.z & kFixedBit)) tround = mark_round(ld(&P.mark[lk.z].v));
            }
            const bool tfix = (lk.z & kFixedBit) != 0;
            const int32_t twin = (int32_t)(lk.z & kEdgeMask);
            const bool kill = kills(has, e, twin, tround, now);
            BloomRec *const B = &P.bloom[lk.y];
            u64 old = 1;
            if (kill) {
                old = atomicAdd(&B->kc, (u64)1);
                st(&P.dead[lk.x], (uint8_t)1);
            }
            const int32_t kb = (int32_t)(old >> 32), d = kb - 1;
            const bool dec = kill && d > 0 && !tfix && tround != now;
            // The first kill of the round queues the bloom; the first of the
            // part records the bloom's number as the part finds it.
            const bool first = kill && d > 0 && (uint32_t)old == 0;
            int32_t otw = 0;
            uint2 w01 = make_uint2(0, 0);
            if (dec) otw = atomicSub(&P.sup[twin], d);
            if (first) {
                w01 = *reinterpret_cast<const uint2 *>(&B->w0);
                if (F != kOne && ld(&B->part) != part) {
                    st(&B->part, part);
                    if (F == kSplit) P.wedge_k[lk.x] = kb;
                }
            }
            const int32_t level = __shfl(level_l.x, src, kWave);
            const bool tf = dec && otw > level && otw - d <= level;
            if (F != kSplit) {
                const int32_t t = __shfl(level_l.y, src, kWave);
                list_edges(P, dec && otw >= t && otw - d < t && otw - d > level, part, twin);
            }
            if (__ballot(first || tf)) {
                uint32_t tlo = 0, thi = 0;
                if (tf) {
                    tlo = (uint32_t)P.link_off[twin];
                    thi = (uint32_t)P.link_off[(int64_t)twin + 1];
                }
                const uint32_t nch = (w01.y - w01.x + kWedgeChunk - 1) / kWedgeChunk;
                const uint32_t tk = chunks_of(tlo, thi);
                const uint32_t ib = wave_inclusive_sum<uint32_t>(nch);
                const uint32_t jf = wave_inclusive_sum<uint32_t>(tk);
                Slots sb, sf;
                reserve2(rb, wave_last(ib), &C->ntc[p].v, rf, wave_last(jf), &C->nf[q].v, grow, sb,
                         sf);
                put_blooms(P.tc[p], sb, nch, ib - nch, (int32_t)lk.y, w01.x);
                put_fronts<F>(P, P.front[q], sf, tf, tk, jf - tk, twin, part, level, now + 1, tlo, thi);
                set_front_flags<F>(P, tf, part, q, flagged);
            }
            upd += dec ? 1 : 0;
        }
    }
    fill_blooms(P.tc[p], rb);
    fill_fronts(P.front[q], rf);
}

// A wedge's two edges lose the kills c of its bloom (lanes with da, db): whether
// they cross the level (f), and level by level the threshold t.
template <SweepForm F, bool UNIT>
__device__ __forceinline__ void take_kills(const SweepArgs &P, bool da, bool db, int32_t ea, int32_t eb,
                                           int32_t c, int32_t level, int32_t t, bool &f1, bool &f2,
                                           bool &t1, bool &t2) {
    f1 = f2 = t1 = t2 = false;
    if (UNIT) {
        // Ablation: one unit per kill; the step from level + 1 crosses (from
        // the threshold, crosses that).  A sweep's blooms lose many wedges a
        // round, so eight kills' atomics are in flight together (5M-edge graph
        // 1,780 -> 668 ms).
        constexpr int kUnits = 8;
        for (int32_t x = 0; x < (da || db ? c : 0); x += kUnits) {
            int32_t o1[kUnits], o2[kUnits];
#pragma unroll
            for (int k = 0; k < kUnits; ++k) {
                o1[k] = o2[k] = -1;
                if (da && x + k < c) o1[k] = atomicSub(&P.sup[ea], 1);
                if (db && x + k < c) o2[k] = atomicSub(&P.sup[eb], 1);
            }
#pragma unroll
            for (int k = 0; k < kUnits; ++k) {
                f1 |= da && x + k < c && o1[k] == level + 1;
                f2 |= db && x + k < c && o2[k] == level + 1;
                if (F != kSplit) {
                    t1 |= da && x + k < c && o1[k] == t;
                    t2 |= db && x + k < c && o2[k] == t;
                }
            }
        }
    } else {
        int32_t o1 = 0, o2 = 0;
        if (da) o1 = atomicSub(&P.sup[ea], c);
        if (db) o2 = atomicSub(&P.sup[eb], c);
        f1 = da && o1 > level && o1 - c <= level;
        f2 = db && o2 > level && o2 - c <= level;
        if (F != kSplit) {
            t1 = da && o1 >= t && o1 - c < t && o1 - c > level;
            t2 = db && o2 >= t && o2 - c < t && o2 - c > level;
        }
    }
}

// Phase B likewise.
template <bool UNIT>
__device__ __forceinline__ void sweep_phase_b_few(const SweepArgs &P, int64_t r, int p, u64 ntc,
                                                  int2 one, int64_t wid, int64_t nwaves,
                                                  uint32_t &upd, uint32_t &visits, uint32_t &touch,
                                                  uint32_t &unb) {
    SweepCtl *C = P.ctl;
    const int q = p ^ 1;
    const int32_t level = one.x, thresh = one.y;
    const u64 *const items = reinterpret_cast<const u64 *>(P.tc[p]);
    bool flagged = false;
    u64 item = 0;
    if (wid < (int64_t)ntc) item = ld(&items[wid]);
    for (int64_t i = wid; i < (int64_t)ntc; i += nwaves) {
        const u64 cur = item;
        if (i + nwaves < (int64_t)ntc) item = ld(&items[i + nwaves]);  // loaded early
        const int32_t b = (int32_t)(uint32_t)cur;
        if (b < 0) continue;
        BloomRec *const B = &P.bloom[b];
        const uint32_t w = (uint32_t)(cur >> 32) + lane_id();
        const u64 kc = ld(&B->kc);
        const uint2 w01 = *reinterpret_cast<const uint2 *>(&B->w0);
        // The piece's end is not known yet: its loads stay below the index's
        // end, and what lies past the bloom's is left out.
        const uint32_t at = min(w, P.n_w);
        const uint32_t ra = (uint32_t)P.wea[at], rb = (uint32_t)P.web[at];
        const uint8_t gone = ld(&P.dead[at]);
        const int32_t c = (int32_t)(uint32_t)kc, kn = (int32_t)(kc >> 32) - c;
        const uint32_t nch = (w01.y - w01.x + kWedgeChunk - 1) / kWedgeChunk;
        const bool live = w < w01.y && kn > 0 && !gone;
        const bool da = live && !(ra & kFixedBit), db = live && !(rb & kFixedBit);
        const int32_t ea = (int32_t)(ra & kEdgeMask), eb = (int32_t)(rb & kEdgeMask);
        uint32_t lo1 = 0, hi1 = 0, lo2 = 0, hi2 = 0;
        if (da) {
            lo1 = (uint32_t)P.link_off[ea];
            hi1 = (uint32_t)P.link_off[(int64_t)ea + 1];
        }
        if (db) {
            lo2 = (uint32_t)P.link_off[eb];
            hi2 = (uint32_t)P.link_off[(int64_t)eb + 1];
        }
        bool f1, f2, t1, t2;
        take_kills<kOne, UNIT>(P, da, db, ea, eb, c, level, thresh, f1, f2, t1, t2);
        if (__ballot(f1 || f2)) {
            const uint32_t k1 = f1 ? chunks_of(lo1, hi1) : 0u, k2 = f2 ? chunks_of(lo2, hi2) : 0u;
            u64 base[3];
            wave_alloc3(k1 + k2, &C->nf[q].v, 0u, nullptr, 0u, nullptr, base);
            const Slots S{0, 0, 0xffffffffu};
            put_fronts<kOne>(P, P.front[q], S, f1, k1, (uint32_t)base[0], ea, 0, level,
                             (int32_t)(r + 1), lo1, hi1);
            put_fronts<kOne>(P, P.front[q], S, f2, k2, (uint32_t)base[0] + k1, eb, 0, level,
                             (int32_t)(r + 1), lo2, hi2);
            if (!flagged && lane_id() == 0) set_front_flag(P, 0, q);
            flagged = true;
        }
        list_edges(P, t1, 0, ea);
        list_edges(P, t2, 0, eb);
        const int32_t each = UNIT ? c : 1;
        upd += (uint32_t)((da ? each : 0) + (db ? each : 0));
        if (!UNIT) unb += (uint32_t)((da ? c - 1 : 0) + (db ? c - 1 : 0));
        touch += live ? 1 : 0;
        // (See sweep_phase_b.)
        if (lane_id() == 0 && kn != INT_MIN &&
            (nch == 1 || atomicAdd(&B->done, 1) == (int32_t)nch - 1)) {
            st(&B->kc, (u64)(uint32_t)kn << 32);
            if (nch > 1) st(&B->done, 0);
            visits += 1;
        }
    }
}

// Phase B: the survivors of every touched bloom lose its kills; the last
// chunk of a bloom to finish settles it.  Then the round's gathers.
template <SweepForm F, bool UNIT>
__device__ __forceinline__ void sweep_phase_b(const SweepArgs &P, int64_t r, int p, u64 ntc, u64 ngth, int2 one,
                                              int64_t wid, int64_t nwaves, u64 *mask, uint32_t &upd,
                                              uint32_t &visits, uint32_t &touch, uint32_t &unb) {
    SweepCtl *C = P.ctl;
    const int q = p ^ 1;
    const uint32_t per = items_per_step(ntc, nwaves, P.short_b);
    const uint32_t grow = per > 1 ? min(2 * per, P.reserve) : 0u;
    Reserve rf;
    int32_t flagged = -1;
    const bool few = F == kOne && per == 1;
    if (few) sweep_phase_b_few<UNIT>(P, r, p, ntc, one, wid, nwaves, upd, visits, touch, unb);
    for (int64_t g0 = wid * per; !few && g0 < (int64_t)ntc; g0 += nwaves * per) {
        const bool ok = (uint32_t)lane_id() < per && g0 + lane_id() < (int64_t)ntc;
        int32_t b_l = -1, part_l = 0, c_l = 0, k_l = 0;
        int2 level_l = make_int2(0, 0);
        uint32_t lo_l = P.n_w, n = ok ? 1u : 0u, nch = 0;
        if (ok) {
            const u64 item = ld(reinterpret_cast<const u64 *>(&P.tc[p][g0 + lane_id()]));
            b_l = (int32_t)(uint32_t)item;
            if (b_l >= 0) {
                const BloomRec *B = &P.bloom[b_l];
                const u64 kc = ld(&B->kc);
                const uint2 w01 = *reinterpret_cast<const uint2 *>(&B->w0);
                part_l = F == kOne ? 0 : ld(&B->part);
                c_l = (int32_t)(uint32_t)kc;
                k_l = (int32_t)(kc >> 32);
                lo_l = (uint32_t)(item >> 32);
                n = min(w01.y - lo_l, (uint32_t)kWedgeChunk);
                nch = (w01.y - w01.x + kWedgeChunk - 1) / kWedgeChunk;
                level_l = part_level<F>(P, part_l, one);
            }
        }
        const uint32_t inc = wave_inclusive_sum<uint32_t>(n);
        const uint32_t start = inc - n;
        const uint32_t total = wave_last(inc);
        for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
            const int src = per == 1 ? 0 : item_of(ok, start, t0, mask);
            const uint32_t x = t0 + lane_id();
            const bool inr = x < total;
            const uint32_t w = __shfl(lo_l - start, src, kWave) + x;
            uint32_t ra = kFixedBit, rb = kFixedBit;
            uint8_t gone = 1;
            if (inr) {
                ra = (uint32_t)P.wea[w];
                rb = (uint32_t)P.web[w];
                gone = ld(&P.dead[w]);
            }
            const int32_t part = __shfl(part_l, src, kWave);
            const int32_t c = __shfl(c_l, src, kWave), kn = __shfl(k_l, src, kWave) - c;
            const bool live = kn > 0 && !gone;
            const bool da = live && !(ra & kFixedBit), db = live && !(rb & kFixedBit);
            const int32_t ea = (int32_t)(ra & kEdgeMask), eb = (int32_t)(rb & kEdgeMask);
            const int32_t level = __shfl(level_l.x, src, kWave);
            const int32_t t = F != kSplit ? __shfl(level_l.y, src, kWave) : 0;
            bool f1, f2, t1, t2;
            take_kills<F, UNIT>(P, da, db, ea, eb, c, level, t, f1, f2, t1, t2);
            if (F != kSplit) {
                list_edges(P, t1, part, ea);
                list_edges(P, t2, part, eb);
            }
            if (__ballot(f1 || f2)) {
                uint32_t lo1 = 0, hi1 = 0, lo2 = 0, hi2 = 0;
                if (f1) {
                    lo1 = (uint32_t)P.link_off[ea];
                    hi1 = (uint32_t)P.link_off[(int64_t)ea + 1];
                }
                if (f2) {
                    lo2 = (uint32_t)P.link_off[eb];
                    hi2 = (uint32_t)P.link_off[(int64_t)eb + 1];
                }
                const uint32_t k1 = chunks_of(lo1, hi1), k2 = chunks_of(lo2, hi2);
                const uint32_t i1 = wave_inclusive_sum<uint32_t>(k1 + k2);
                Slots sf, none;
                Reserve no;
                reserve2(rf, wave_last(i1), &C->nf[q].v, no, 0u, nullptr, grow, sf, none);
                put_fronts<F>(P, P.front[q], sf, f1, k1, i1 - k1 - k2, ea, part, level, (int32_t)(r + 1),
                           lo1, hi1);
                put_fronts<F>(P, P.front[q], sf, f2, k2, i1 - k2, eb, part, level, (int32_t)(r + 1), lo2,
                           hi2);
                set_front_flags<F>(P, f1 || f2, part, q, flagged);
            }
            const int32_t each = UNIT ? c : 1;
            upd += (uint32_t)((da ? each : 0) + (db ? each : 0));
            if (!UNIT) unb += (uint32_t)((da ? c - 1 : 0) + (db ? c - 1 : 0));
            touch += live ? 1 : 0;
        }
        // A chunk counts itself done once its reads of the bloom's counts
        // have returned (they are used above), so the last one's update of
        // both cannot overtake them.
        if (b_l >= 0) {
            const int32_t kn = k_l - c_l;
            BloomRec *B = &P.bloom[b_l];
            if (kn != INT_MIN && (nch == 1 || atomicAdd(&B->done, 1) == (int32_t)nch - 1)) {
                st(&B->kc, (u64)(uint32_t)kn << 32);
                if (nch > 1) st(&B->done, 0);
                visits += 1;
            }
        }
    }
    fill_fronts(P.front[q], rf);
    int32_t mn_job = -1, mn_all = INT_MAX;
    for (int64_t i = wid; i < (int64_t)ngth; i += nwaves)
        sweep_gather<F>(P, r, p, ld_item(&P.gth[p][i]), mn_job, mn_all, flagged);
    flush_min(P, p, mn_job, mn_all);
}

// Adds the lanes' statistics to the control block and clears them.
__device__ __forceinline__ void sweep_flush(SweepCtl *C, uint32_t &upd, uint32_t &visits,
                                            uint32_t &touch, uint32_t &unb) {
    const u64 a = wave_sum<u64>(upd), b = wave_sum<u64>(visits), c = wave_sum<u64>(touch),
              d = wave_sum<u64>(unb);
    if (lane_id() == 0) {
        if (a) atomicAdd(&C->updates.v, a);
        if (b) atomicAdd(&C->bloom_visits.v, b);
        if (c) atomicAdd(&C->touched.v, c);
        if (d) atomicAdd(&C->unbatched.v, d);
    }
    upd = visits = touch = unb = 0;
}

template <SweepForm F, bool UNIT>
__global__ __launch_bounds__(kPBlock) void k_sweep(SweepArgs P, GridBar *B, int64_t max_rounds,
                                                   int prof) {
    SweepCtl *C = P.ctl;
    __shared__ u64 s_nf, s_ngth, s_nsel, s_ntc, s_left, s_r0;
    __shared__ int s_ok, s_y;
    __shared__ int2 s_level;  // of the only job (level by level; else -1)
    __shared__ u64 s_mask[kPBlock / kWave];
    __shared__ const int32_t *s_ys;
    u64 gen_local = 0;
    // Wave ids run across blocks first: a small round spreads over many CUs.
    const int64_t wid = (int64_t)(threadIdx.x / kWave) * gridDim.x + blockIdx.x;
    const int64_t nwaves = (int64_t)gridDim.x * (kPBlock / kWave);
    // Decisions are made by the last waves, as phase A's items go to the first
    // ones (a round of few items is a chain of waits for memory).
    const int64_t tid = (nwaves - 1 - wid) * kWave + lane_id();
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    uint32_t upd = 0, visits = 0, touch = 0, unb = 0;
    if (threadIdx.x == 0) {
        // A launch resumes at the round where the previous one yielded.
        s_r0 = ld(&C->rounds);
        s_left = 1;  // a launch has something to do (see below)
        s_nf = ld(&C->nf[s_r0 & 1].v);
        const int2 none = make_int2(-1, 0);
        s_level = F == kOne ? part_level<kMany>(P, 0, none) : none;
        s_nsel = ld(&C->nsel[s_r0 & 1].v) & ~kYieldBit;
        s_ys = reinterpret_cast<const int32_t *>(ld(&C->yield_src));
        s_ok = 1;
        s_y = 0;
    }
    u64 looked = tid == 0 ? wall_clock64() : 0;  // at the yield word
    if (lead) st(&C->yielded, 0);
    __syncthreads();
    int64_t r = (int64_t)s_r0;
    for (; r < max_rounds && s_left > 0 && s_ok; ++r) {
        const int p = (int)(r & 1), q = p ^ 1;
        const u64 nf = s_nf, nsel = s_nsel;
        // It changes in rounds without a frontier only (gathers read it anew).
        const int2 one = s_level;
        u64 t0 = 0, t1 = 0, t2 = 0, t3 = 0, t4 = 0;
        if (prof && lead) t0 = wall_clock64();
        if (lead) {
            st(&C->ntc[q].v, (u64)0);
            st(&C->ngth[q].v, (u64)0);
        }
        // The host's yield word is passed on before a barrier and read by every
        // block after it, so all blocks stop after the same round.  One of the
        // last waves looks, which have no items in small rounds: the read takes
        // about 2 us.
        if (tid == 0 && s_ys &&
            (r % kYieldEvery == kYieldEvery - 1 || wall_clock64() - looked >= kYieldTicks)) {
            if (__hip_atomic_load(s_ys, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM))
                atomicOr(&C->nsel[q].v, kYieldBit);
            looked = wall_clock64();
        }
        sweep_decide<F>(P, r, p, tid, nwaves * kWave);
        // Selects take their blocks out of phase A (they are chains of waits
        // behind its traffic), unless there are too many.
        const u64 busy = nsel <= gridDim.x / 2 ? nsel : 0;
        for (u64 i = blockIdx.x; F == kSplit && i < nsel; i += gridDim.x)
            sweep_select(P, ld(&P.sel[p][i]), r, p);
        if (prof && lead) t1 = wall_clock64();
        if (blockIdx.x >= busy)
            sweep_phase_a<F>(P, r, p, nf, one,
                          (int64_t)(threadIdx.x / kWave) * (gridDim.x - busy) + blockIdx.x - busy,
                          (int64_t)(gridDim.x - busy) * (kPBlock / kWave),
                          &s_mask[threadIdx.x / kWave], upd);
        if (prof && lead) t2 = wall_clock64();
        drain_memory();
        __syncthreads();
        if (threadIdx.x == 0) {
            s_ok = grid_arrive_wait(B, gen_local);
            s_ntc = ld(&C->ntc[p].v);
            s_ngth = ld(&C->ngth[p].v);
            // Jobs end in sweep_decide alone, so this count is the same for
            // every block between the round's barriers.  Past the second one a
            // faster block may already decide on the next round: a block that
            // read 0 there would leave while others wait for it.
            s_left = ld(&C->left.v);
        }
        __syncthreads();
        if (!s_ok) break;
        if (prof && lead) t3 = wall_clock64();
        if (lead) {
            st(&C->nf[p].v, (u64)0);
            st(&C->nsel[p].v, (u64)0);
        }
        sweep_phase_b<F, UNIT>(P, r, p, s_ntc, s_ngth, one, wid, nwaves, &s_mask[threadIdx.x / kWave], upd, visits, touch,
                      unb);
        drain_memory();
        __syncthreads();
        if (threadIdx.x == 0) {
            s_ok = grid_arrive_wait(B, gen_local);
            s_nf = ld(&C->nf[q].v);
            if (F == kOne) s_level = part_level<kMany>(P, 0, make_int2(-1, 0));
            const u64 ns = ld(&C->nsel[q].v);
            s_nsel = ns & ~kYieldBit;
            s_y = s_ok && (ns & kYieldBit) != 0;
        }
        __syncthreads();
        if (prof && lead) {
            t4 = wall_clock64();
            C->prof[0] += t1 - t0;
            C->prof[1] += t2 - t1;
            C->prof[2] += t3 - t2;
            C->prof[3] += t4 - t3;
        }
        if ((r & 1023) == 1023) sweep_flush(C, upd, visits, touch, unb);  // 32-bit per lane
        if (s_y) {
            ++r;
            if (lead && s_left > 0) st(&C->yielded, 1);
            break;
        }
    }
    sweep_flush(C, upd, visits, touch, unb);
    if (lead) st(&C->rounds, (u64)r);
}

// The same rounds as two kernels each, replayed from a captured HIP graph or
// launched directly (a job list that is done makes them empty).
template <SweepForm F>
__global__ __launch_bounds__(kPBlock) void k_sweep_a(SweepArgs P, int p) {
    SweepCtl *C = P.ctl;
    __shared__ u64 s_r, s_nf, s_nsel, s_mask[kPBlock / kWave];
    if (threadIdx.x == 0) {
        s_r = ld(&C->rounds);
        s_nf = ld(&C->nf[p].v);
        s_nsel = ld(&C->nsel[p].v);
    }
    __syncthreads();
    const int q = p ^ 1;
    const int64_t wid = (int64_t)(threadIdx.x / kWave) * gridDim.x + blockIdx.x;
    const int64_t nwaves = (int64_t)gridDim.x * (kPBlock / kWave);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st(&C->ntc[q].v, (u64)0);
        st(&C->ngth[q].v, (u64)0);
        st(&C->round_b, s_r);
    }
    sweep_decide<F>(P, (int64_t)s_r, p, (nwaves - 1 - wid) * kWave + lane_id(), nwaves * kWave);
    for (u64 i = blockIdx.x; F == kSplit && i < s_nsel; i += gridDim.x)
        sweep_select(P, ld(&P.sel[p][i]), (int64_t)s_r, p);
    uint32_t upd = 0, none = 0;
    sweep_phase_a<F>(P, (int64_t)s_r, p, s_nf, make_int2(-1, 0), wid, nwaves, &s_mask[threadIdx.x / kWave], upd);
    sweep_flush(C, upd, none, none, none);
}

template <SweepForm F, bool UNIT>
__global__ __launch_bounds__(kPBlock) void k_sweep_b(SweepArgs P, int p) {
    SweepCtl *C = P.ctl;
    __shared__ u64 s_ntc, s_ngth, s_r, s_mask[kPBlock / kWave];
    if (threadIdx.x == 0) {
        s_ntc = ld(&C->ntc[p].v);
        s_ngth = ld(&C->ngth[p].v);
        s_r = ld(&C->round_b);
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st(&C->nf[p].v, (u64)0);
        st(&C->nsel[p].v, (u64)0);
        // Phase B reads round_b, phase A rounds: each is set where the other
        // kernel runs.
        if (ld(&C->left.v) > 0) st(&C->rounds, s_r + 1);
    }
    uint32_t upd = 0, visits = 0, touch = 0, unb = 0;
    sweep_phase_b<F, UNIT>(P, (int64_t)s_r, p, s_ntc, s_ngth, make_int2(-1, 0), (int64_t)(threadIdx.x / kWave) * gridDim.x + blockIdx.x,
                  (int64_t)gridDim.x * (kPBlock / kWave), &s_mask[threadIdx.x / kWave], upd, visits,
                  touch, unb);
    sweep_flush(C, upd, visits, touch, unb);
}

// Edge and bloom state at a sweep's start.  Edges fixed by earlier passes
// (progressive mode) are in no part and never taken: their support is out of
// reach.
__global__ void k_sweep_edges(const uint64_t *supl, int64_t m, const int32_t *fixed, int32_t *sup,
                              EdgeMark *mark, int64_t *sup_out) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = (int32_t)(supl[e] & 0xffffffffu);
        const bool fx = fixed && fixed[e];
        sup[e] = fx ? INT_MAX : v;
        mark[e].v = edge_mark(fx ? INT_MAX : -1, INT_MAX);
        if (sup_out) sup_out[e] = v;
    }
}

__global__ void k_put_byte(uint8_t *p, uint8_t v) { *p = v; }

__global__ void k_sweep_blooms(const uint32_t *bwoff, const int32_t *bk, int64_t n, BloomRec *rec) {
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < n;
         b += (int64_t)gridDim.x * blockDim.x)
        rec[b] = BloomRec{(u64)(uint32_t)bk[b] << 32, bwoff[b], bwoff[b + 1], -1, 0};
}

// Captured chunks of rounds, cached in the workspace by argument bytes.
template <typename F>
hipGraphExec_t chunk_graph(const void *args, size_t bytes, int rounds, Workspace &ws, F &&launch) {
    const unsigned char *a = static_cast<const unsigned char *>(args);
    std::vector<unsigned char> key(a, a + bytes);
    auto &cache = ws.graphs;
    for (auto &g : cache)
        if (g.rounds == rounds && g.key == key) return g.exec;
    if (cache.size() >= 16) {
        (void)hipGraphExecDestroy(cache.front().exec);
        cache.erase(cache.begin());
    }
    hipStream_t cs;
    BT_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipGraph_t g;
    BT_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    launch(cs);
    BT_HIP(hipStreamEndCapture(cs, &g));
    hipGraphExec_t ex;
    BT_HIP(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0));
    (void)hipGraphDestroy(g);
    (void)hipStreamDestroy(cs);
    cache.push_back(Workspace::GraphEntry{key, rounds, ex});
    return ex;
}

// Parts each job of n edges aims at in a sweep: fewer parts touch each bloom
// less often, more leave less to deeper sweeps.  Of caps of 4, 8, 12, 16, 24,
// 32, 48 and 64 the 5M-edge graph took 316, 262, 258, 245, 240, 238, 260 and
// 286 ms, 1,024 pool graphs 1541, 1324, 1237, 1205, 1162, 1211, 1287 and 1347
// ms; a 200k-edge graph, bound by its leaves' rounds, takes 32 best.
int64_t parts_for(int64_t n, int64_t work, int64_t total) {
    const int64_t cap = total >= (int64_t(1) << 20) ? 24 : 32;
    return std::max<int64_t>(4, std::min<int64_t>(cap, std::max<int64_t>(n / 2048, work / 32768)));
}

// What a sweep is asked: supl holds the jobs' supports; progressive passes
// carry fixed edges and a first level.
struct SweepAsk {
    const uint64_t *supl = nullptr;
    const int32_t *fixed = nullptr;
    int32_t min_level = 0;
    bool unit = false, plain = false;
    bool least = false;          // with the least memory
    int64_t *sup_out = nullptr;
    int64_t *scratch = nullptr;  // plain: m words that the caller writes afterwards
};

// The state of a sweep over one job.
__global__ void k_sweep_init(SweepArgs P, JobState job, SplitPart first, int32_t n_parts,
                             u64 yield_src) {
    u64 *c = reinterpret_cast<u64 *>(P.ctl);
    for (uint32_t i = threadIdx.x; i < sizeof(SweepCtl) / sizeof(u64); i += blockDim.x) c[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        P.ctl->left.v = 1;
        P.ctl->n_parts.v = (u64)n_parts;
        P.ctl->yield_src = yield_src;
        P.js[0] = job;
        if (n_parts) P.parts[0] = first;
    }
}

// State of a sweep over the jobs of a depth, ready for its first round by
// `pblocks` workgroups.
SweepArgs sweep_setup(const SplitIndex &ix, const std::vector<SplitJob> &jobs, const SweepAsk &ask,
                      int pblocks, const int32_t *yield_word, Workspace &ws, hipStream_t s) {
    const int64_t m = ix.m;
    const int32_t nj = (int32_t)jobs.size();
    if (2 * ix.n_w >= (int64_t)UINT32_MAX)
        throw Error{BT_EOVERFLOW, "edge-to-wedge links must be below 2^32"};
    const int64_t nb = ix.n_b > 0 ? ix.n_b : 1;
    // A round's frontier list takes the slots that two phases leave over.
    const int64_t waves = (int64_t)pblocks * (kPBlock / kWave);
    const int64_t spare = spare_slots(m, waves, ask.least);
    const int64_t max_tc = nb + ix.n_w / kWedgeChunk + 1 + spare;
    const int64_t max_front = m + 2 * ix.n_w / kLinkChunk + 1 + 2 * spare;
    const int64_t max_gth = m / kGatherChunk + nj + 1;
    const int64_t max_parts = ask.plain ? nj : (int64_t)nj * (kMaxParts + 1) + 1;
    SweepArgs P{};
    P.ctl = ws.get<SweepCtl>("sw_ctl", 1);
    P.js = ws.get<JobState>("sw_jobs", nj);
    P.n_jobs = nj;
    P.parts = ws.get<SplitPart>("sw_parts", max_parts);
    P.sup = ws.get<int32_t>("peel_sup", m);
    P.mark = ws.get<EdgeMark>("sw_mark", m);
    const int64_t dead_bytes = (ix.n_w + 4) & ~int64_t(3);
    P.dead = ws.get<uint8_t>("sw_dead", dead_bytes);
    P.bloom = ws.get<BloomRec>("sw_bloom", nb);
    P.wedge_k = ask.plain ? nullptr : ws.get<int32_t>("sw_wedge_k", ix.n_w);
    // Links of an edge, wedges of a bloom, on average.
    const int64_t links = 2 * ix.n_w / m + 1, wedges = ix.n_w / nb + 1;
    P.short_a = links <= 16 ? (int32_t)(kWave / links) : 0;
    P.short_b = wedges <= 3 ? (int32_t)(kWave / wedges) : 0;
    P.list = reinterpret_cast<int32_t *>(ask.scratch);
    P.wea = ix.wea;
    P.web = ix.web;
    P.link_off = ix.link_off;
    P.link = ix.link;
    P.n_w = (uint32_t)ix.n_w;
    P.reserve = (uint32_t)(spare / waves);
    P.front[0] = ws.get<FrontItem>("peel_front0", max_front);
    P.front[1] = ws.get<FrontItem>("peel_front1", max_front);
    P.tc[0] = ws.get<SweepBloomItem>("peel_tc0", max_tc);
    P.tc[1] = ws.get<SweepBloomItem>("peel_tc1", max_tc);
    P.gth[0] = ws.get<SweepGatherItem>("sw_gth0", max_gth);
    P.gth[1] = ws.get<SweepGatherItem>("sw_gth1", max_gth);
    P.sel[0] = ws.get<int32_t>("sw_sel0", nj);
    P.sel[1] = ws.get<int32_t>("sw_sel1", nj);

    k_sweep_edges<<<grid_for(m, 256, 16384), 256, 0, s>>>(ask.supl, m, ask.fixed, P.sup, P.mark,
                                                         ask.sup_out);
    BT_CHECK_LAUNCH();
    if (ix.n_b > 0) {
        k_sweep_blooms<<<grid_for(ix.n_b, 256, 16384), 256, 0, s>>>(ix.bwoff, ix.bk, ix.n_b, P.bloom);
        BT_CHECK_LAUNCH();
    }
    zero_bytes(P.dead, (size_t)dead_bytes, s);
    k_put_byte<<<1, 1, 0, s>>>(P.dead + ix.n_w, 1);  // the null items' wedge
    BT_CHECK_LAUNCH();
    if (ix.n_w && !ask.plain) zero_bytes(P.wedge_k, sizeof(int32_t) * ix.n_w, s);

    std::vector<JobState> js((size_t)nj);
    std::vector<SplitPart> first((size_t)nj);
    // Progressive passes begin with a part at min_level: the edges outside the
    // pass's bitruss, which need no numbers.
    const bool preset = ask.min_level > 0 || ask.plain;
    for (int32_t j = 0; j < nj; ++j) {
        JobState &J = js[(size_t)j];
        std::memset(&J, 0, sizeof J);
        J.state = kJobActive;
        J.e0 = jobs[(size_t)j].e0;
        J.e1 = J.e0 + jobs[(size_t)j].ne;
        J.gmin[0] = INT_MAX;
        J.gmin[1] = preset ? ask.min_level : INT_MAX;
        J.gather_round = preset ? -1 : -8;
        J.select_round = -8;
        J.level = -1;
        J.part = j;
        J.thresh = -1;
        J.delta = 7;
        J.scale = 1.f;
        J.narrow = jobs[(size_t)j].stuck ? 1 : 0;
        J.hi_bound = jobs[(size_t)j].hi;
        const int64_t n = jobs[(size_t)j].ne;
        J.target_n = std::max<int64_t>(512, n / parts_for(n, jobs[(size_t)j].work, m));
        first[(size_t)j] = SplitPart{ask.min_level, ask.plain ? INT_MIN : ask.min_level, j, 1};
    }
    if (nj == 1) {
        // By value: copies from the host's arrays and the wait for them took 50
        // us of each of BiT-PC's passes.
        k_sweep_init<<<1, 256, 0, s>>>(P, js[0], first[0], preset ? 1 : 0,
                                       reinterpret_cast<u64>(yield_word));
        BT_CHECK_LAUNCH();
        return P;
    }
    BT_HIP(hipMemcpyAsync(P.js, js.data(), sizeof(JobState) * nj, hipMemcpyHostToDevice, s));
    if (preset)
        BT_HIP(hipMemcpyAsync(P.parts, first.data(), sizeof(SplitPart) * nj, hipMemcpyHostToDevice,
                              s));
    SweepCtl init{};
    init.left.v = (u64)nj;
    init.n_parts.v = preset ? (u64)nj : 0;
    init.yield_src = reinterpret_cast<u64>(yield_word);
    BT_HIP(hipMemcpyAsync(P.ctl, &init, sizeof init, hipMemcpyHostToDevice, s));
    BT_HIP(hipStreamSynchronize(s));  // the host arrays are read until here
    return P;
}

using SweepKernel = void (*)(SweepArgs, GridBar *, int64_t, int);
SweepKernel sweep_kernel(SweepForm form, bool unit) {
    static const SweepKernel k[3][2] = {{k_sweep<kSplit, false>, k_sweep<kSplit, true>},
                                        {k_sweep<kMany, false>, k_sweep<kMany, true>},
                                        {k_sweep<kOne, false>, k_sweep<kOne, true>}};
    return k[form][unit ? 1 : 0];
}

// BT_PEEL_YIELD=1 makes every launch stop at its first check (a test of the
// resume path).
const int32_t *yield_word(const CoopTurn *turn) {
    const char *yv = std::getenv("BT_PEEL_YIELD");
    return turn ? turn->yield_word(yv && std::atoi(yv) == 1) : nullptr;
}

// One sweep over the jobs of a depth; `turn` is held.
SweepResult sweep(const SplitIndex &ix, const std::vector<SplitJob> &jobs, const SweepAsk &ask,
                  const TuneParams &tp, CoopTurn *turn, PeelCounters &pc, Workspace &ws,
                  hipStream_t s) {
    const int64_t m = ix.m;
    const int32_t nj = (int32_t)jobs.size();
    int dev = 0, cus = 0, occ = 0;
    BT_HIP(hipGetDevice(&dev));
    BT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const auto kern = sweep_kernel(ask.plain ? (nj == 1 ? kOne : kMany) : kSplit, ask.unit);
    BT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, kPBlock, 0));
    const int pblocks = !turn ? cus
                        : tp.peel_blocks == 0 && m >= kAllCusEdges
                            ? std::max(1, std::min(cus, occ * cus))
                            : peel_grid(tp, cus, occ * cus);
    SweepArgs P = sweep_setup(ix, jobs, ask, pblocks, yield_word(turn), ws, s);
    hipEvent_t ev0, ev1;
    BT_HIP(hipEventCreate(&ev0));
    BT_HIP(hipEventCreate(&ev1));
    struct EvFree {
        hipEvent_t a, b;
        ~EvFree() {
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
        }
    } ev_free{ev0, ev1};
    SweepCtl hc{};
    const int64_t max_rounds = 8 * m + 1024;
    const int prof = std::getenv("BT_PEEL_PROFILE") ? 1 : 0;
    const bool verbose = std::getenv("BT_PEEL_VERBOSE") != nullptr;
    float ms = 0.f;
    if (turn) {
        GridBar *bar = ws.get<GridBar>("peel_bar", 1);
        void *args[] = {&P, &bar, (void *)&max_rounds, (void *)&prof};
        for (;;) {
            zero_bytes(bar, sizeof(GridBar), s);
            BT_HIP(hipEventRecord(ev0, s));
            BT_HIP(hipLaunchCooperativeKernel((const void *)kern, dim3(pblocks), dim3(kPBlock),
                                              args, 0, s));
            BT_HIP(hipEventRecord(ev1, s));
            int32_t fail = 0;
            char *h = reinterpret_cast<char *>(ws.host((int)(sizeof hc / sizeof(int64_t)) + 1));
            BT_HIP(hipMemcpyAsync(h, P.ctl, sizeof hc, hipMemcpyDeviceToHost, s));
            BT_HIP(hipMemcpyAsync(h + sizeof hc, &bar->fail, sizeof fail, hipMemcpyDeviceToHost, s));
            BT_HIP(hipStreamSynchronize(s));
            std::memcpy(&hc, h, sizeof hc);
            std::memcpy(&fail, h + sizeof hc, sizeof fail);
            float t = 0.f;
            BT_HIP(hipEventElapsedTime(&t, ev0, ev1));
            ms += t;
            if (fail) throw Error{BT_EDEVICE, "peel grid barrier timed out"};
            if (hc.left.v == 0) break;
            if (!hc.yielded) throw Error{BT_EDEVICE, "peel stopped early"};
            // Each launch that yields has run at least one round.
            if ((int64_t)hc.rounds >= max_rounds) throw Error{BT_EDEVICE, "peel made no progress"};
            pc.yields += 1;
            turn->requeue();
        }
    } else {
        const char *gv = std::getenv("BT_PEEL_GRAPH");
        const bool use_graph = !(gv && std::atoi(gv) == 0);
        constexpr int kChunk = 32;
        const auto kern_a = ask.plain ? k_sweep_a<kMany> : k_sweep_a<kSplit>;
        const auto kern_b = ask.plain ? (ask.unit ? k_sweep_b<kMany, true> : k_sweep_b<kMany, false>)
                                      : (ask.unit ? k_sweep_b<kSplit, true> : k_sweep_b<kSplit, false>);
        const auto rounds = [&](hipStream_t t) {
            for (int k = 0; k < kChunk; ++k) {
                kern_a<<<cus, kPBlock, 0, t>>>(P, k & 1);
                kern_b<<<cus, kPBlock, 0, t>>>(P, k & 1);
            }
        };
        hipGraphExec_t ex = nullptr;
        if (use_graph) ex = chunk_graph(&P, sizeof P, kChunk, ws, rounds);
        do {
            BT_HIP(hipEventRecord(ev0, s));
            if (use_graph) {
                BT_HIP(hipGraphLaunch(ex, s));
            } else {
                rounds(s);
                BT_CHECK_LAUNCH();
            }
            BT_HIP(hipEventRecord(ev1, s));
            BT_HIP(hipMemcpyAsync(&hc, P.ctl, sizeof hc, hipMemcpyDeviceToHost, s));
            BT_HIP(hipStreamSynchronize(s));
            float t = 0.f;
            BT_HIP(hipEventElapsedTime(&t, ev0, ev1));
            ms += t;
            if ((int64_t)hc.rounds >= max_rounds) throw Error{BT_EDEVICE, "peel made no progress"};
        } while (hc.left.v != 0);
    }
    pc.kernel_ms += ms;
    pc.rounds += (int64_t)hc.rounds;
    pc.updates += (int64_t)hc.updates.v;
    pc.updates_unbatched += (int64_t)(hc.updates.v + hc.unbatched.v);
    pc.bloom_visits += (int64_t)hc.bloom_visits.v;
    pc.touched += (int64_t)hc.touched.v;
    if (verbose)
        std::fprintf(stderr,
                     "[peel] sweep: %d jobs, %lld edges, %lld blooms, %lld wedges: %.2f ms, %llu rounds, %llu parts, %.3g updates\n",
                     nj, (long long)m, (long long)ix.n_b, (long long)ix.n_w, (double)ms, hc.rounds,
                     hc.n_parts.v, (double)hc.updates.v);
    if (prof)
        std::fprintf(stderr, "[peel] block0 us: decide %.0f phaseA %.0f bar1 %.0f phaseB+bar2 %.0f\n",
                     hc.prof[0] / 100.0, hc.prof[1] / 100.0, hc.prof[2] / 100.0, hc.prof[3] / 100.0);
    return SweepResult{P.mark, P.wedge_k, P.parts, (int32_t)hc.n_parts.v};
}

__global__ void k_marks_out(const EdgeMark *mark, int64_t m, int64_t *out) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x)
        out[e] = mark_part(mark[e].v);
}

__global__ void k_max_mark(const EdgeMark *mark, int64_t m, unsigned long long *out) {
    unsigned long long v = 0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = mark_part(mark[e].v);
        if (p != INT_MAX) v = max(v, (unsigned long long)max(p, 0));  // not the fixed ones
    }
    for (int d = kWave / 2; d > 0; d >>= 1) v = max(v, (unsigned long long)__shfl_xor(v, d, kWave));
    if (lane_id() == 0) atomicMax(out, v);
}

SplitIndex view_of(const IndexArrays &ix, int64_t m) {
    SplitIndex v;
    v.m = m;
    v.n_b = ix.n_b;
    v.n_w = ix.n_w;
    v.bwoff = ix.bwoff;
    v.bk = ix.bk;
    v.wea = ix.wea;
    v.web = ix.web;
    v.wbl = ix.wbl;
    v.link_off = ix.link_off;
    v.link = ix.link;
    return v;
}

__global__ void k_blooms_live(const BloomRec *rec, int64_t n, int32_t *out) {
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < n;
         b += (int64_t)gridDim.x * blockDim.x)
        out[b] = (int32_t)(rec[b].kc >> 32);
}

}  // namespace

// The peel level by level, one round at a time from the host: after each
// round, the edges whose marks name it, the supports and the blooms' live
// wedges.
void peel_trace(IndexArrays &ix, int64_t m, int64_t *phi_out, const PeelTraceFn &trace,
                Workspace &ws, hipStream_t s) {
    if (m == 0) return;
    const std::vector<SplitJob> jobs{SplitJob{0, 0, (int32_t)m, 0, kLevelMax, 0, false}};
    SweepAsk ask;
    ask.supl = ix.supl;
    ask.plain = true;
    ask.scratch = phi_out;
    const int blocks = 64;
    const SweepArgs P = sweep_setup(view_of(ix, m), jobs, ask, blocks, nullptr, ws, s);
    int32_t *live = ws.get<int32_t>("trace_live", ix.n_b);
    SweepCtl hc{};
    std::vector<EdgeMark> mark((size_t)m);
    for (int64_t r = 0;; ++r) {
        if (r > 8 * m + 1024) throw Error{BT_EDEVICE, "peel made no progress"};
        k_sweep_a<kMany><<<blocks, kPBlock, 0, s>>>(P, (int)(r & 1));
        k_sweep_b<kMany, false><<<blocks, kPBlock, 0, s>>>(P, (int)(r & 1));
        BT_CHECK_LAUNCH();
        if (ix.n_b) k_blooms_live<<<grid_for(ix.n_b, 256, 4096), 256, 0, s>>>(P.bloom, ix.n_b, live);
        BT_CHECK_LAUNCH();
        BT_HIP(hipMemcpyAsync(&hc, P.ctl, sizeof hc, hipMemcpyDeviceToHost, s));
        BT_HIP(hipMemcpyAsync(mark.data(), P.mark, sizeof(EdgeMark) * m, hipMemcpyDeviceToHost, s));
        BT_HIP(hipStreamSynchronize(s));
        PeelTraceRound t;
        for (int64_t e = 0; e < m; ++e)
            if ((int32_t)(uint32_t)mark[(size_t)e].v == (int32_t)r) {
                t.level = (int32_t)(mark[(size_t)e].v >> 32);
                t.removed.push_back((int32_t)e);
            }
        if (!t.removed.empty()) {
            t.sup.resize((size_t)m);
            t.bloom_k.resize((size_t)ix.n_b);
            BT_HIP(hipMemcpy(t.sup.data(), P.sup, sizeof(int32_t) * m, hipMemcpyDeviceToHost));
            if (ix.n_b)
                BT_HIP(hipMemcpy(t.bloom_k.data(), live, sizeof(int32_t) * ix.n_b,
                                 hipMemcpyDeviceToHost));
            trace(t);
        }
        if (hc.left.v == 0) break;
    }
    k_marks_out<<<grid_for(m, 256, 16384), 256, 0, s>>>(P.mark, m, phi_out);
    BT_CHECK_LAUNCH();
}

int64_t peel_split_bytes(int64_t m, int64_t n_b, int64_t n_w, int64_t graphs, bool plain) {
    const int64_t spare = spare_slots(m, 256 * 16, plain);  // waves of a card of 256 CUs
    // Sweep: edges, blooms, wedges, work lists.  The deeper sweeps' blooms
    // are parts of the first's, at most one a wedge.
    const int64_t nb = plain ? n_b : std::max(n_b, n_w);
    int64_t t = 12 * m + 24 * nb + n_w + 32 * (m + n_w / 32 + 2 * spare) +
                16 * (nb + n_w / 64 + spare) + 32 * (m / kGatherChunk + graphs) +
                (128 + 8 + 16 * (plain ? 1 : kMaxParts + 1)) * graphs;
    if (!plain) {
        t += 4 * n_w;                                  // wedge_k
        t += 44 * m + 4 * n_w + 12 * n_w;              // regroup: edges, parts, sort scratch
        t += 2 * (12 * n_w + 8 * nb) + 24 * n_w + 24 * m;  // next depths, their links
        t += 16 * n_w + 8 * nb + 16 * (2 * m + n_w / 32) + 8 * (nb + n_w / 64 + m) + 8 * m;  // leaves
    }
    t += 64 * 256 + 4096;
    return t + t / 8;
}

// Whether a peel of at most so many levels goes level by level.  A level costs
// some 30 us in rounds of its own; a split costs 0.2 ms and more in launches,
// and 0.5 ns a wedge for the first sweep (which a graph of few levels falls
// to as a whole) and the regrouping.  Uniform graphs of 17,000, 117,248,
// 400,000, 1.5M and 4M edges (largest supports 8, 22, 58, about 150 and 350)
// take 0.79, 2.8, 9.8, 41.9 and 190 ms split and 0.55, 2.4, 5.2, 21.7 and 88 ms
// level by level; a Chung-Lu graph of 20,000 edges (thousands) 4.1 and 11.6 ms.
// BT_PEEL_MODE=split splits whatever the levels.
bool few_levels(int64_t levels, int64_t n_w) {
    const char *mv = std::getenv("BT_PEEL_MODE");
    if (mv && std::strcmp(mv, "split") == 0) return false;
    return levels <= 24 + n_w / 65536;
}

const char *const kSplitBuffers[] = {"sw_wedge_k", "rg_", "sp_", "lf_", "pool_", "rs_", nullptr};

// The peel level by level.
static void peel_levels(const SplitIndex &cur, const std::vector<SplitJob> &jobs, const SweepAsk &ask,
                        const TuneParams &tp, CoopTurn *turn, int64_t *phi_out, PeelCounters &pc,
                        Workspace &ws, hipStream_t s) {
    const int64_t m = cur.m;
    // Level by level, with the memory of the index alone.
    const SweepResult sw = sweep(cur, jobs, ask, tp, turn, pc, ws, s);
    k_marks_out<<<grid_for(m, 256, 16384), 256, 0, s>>>(sw.mark, m, phi_out);
    BT_CHECK_LAUNCH();
    unsigned long long *mx = ws.get<unsigned long long>("sp_max", 1);
    zero_bytes(mx, sizeof *mx, s);
    k_max_mark<<<grid_for(m, 256, 4096), 256, 0, s>>>(sw.mark, m, mx);
    BT_CHECK_LAUNCH();
    static_assert(sizeof(JobState) % sizeof(int64_t) == 0, "copied as words");
    int64_t *h = ws.host(1 + (int)(jobs.size() * (sizeof(JobState) / sizeof(int64_t))));
    BT_HIP(hipMemcpyAsync(h, mx, sizeof *mx, hipMemcpyDeviceToHost, s));
    BT_HIP(hipMemcpyAsync(h + 1, ws.get<JobState>("sw_jobs", (int64_t)jobs.size()),
                          sizeof(JobState) * jobs.size(), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    pc.launches += 1 + pc.yields;
    pc.max_phi = h[0];
    const JobState *js = reinterpret_cast<const JobState *>(h + 1);
    for (size_t j = 0; j < jobs.size(); ++j)
        pc.levels = std::max<int64_t>(pc.levels, js[j].n_parts);
}

// The peel that splits; the index's links are lost.
static void peel_parts(const IndexArrays &ix, SplitIndex cur, std::vector<SplitJob> jobs, SweepAsk ask,
                       int32_t ng, const TuneParams &tp, bool coop, CoopTurn *turn, int64_t *phi_out,
                       PeelCounters &pc, Workspace &ws, hipStream_t s) {
    const int64_t m = cur.m;
    const bool verbose = std::getenv("BT_PEEL_VERBOSE") != nullptr;
    std::vector<int32_t> levels((size_t)ng, 0);
    int32_t max_level = 0;
    LeafPool pool;
    std::unique_ptr<LeafRun> leaves;
    int dev = 0, cus = 0;
    BT_HIP(hipGetDevice(&dev));
    BT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    for (int depth = 0; !jobs.empty(); ++depth) {
        const SweepResult sw = sweep(cur, jobs, ask, tp, turn, pc, ws, s);
        // The links are not needed after the first sweep; their memory (24
        // bytes a wedge) takes the leaves' wedges and blooms (20).
        if (depth == 0) pool.place(ix.link, ix.n_w, m, ws);
        Regrouped g;
        regroup(cur, sw, jobs, depth, phi_out, levels, max_level, g, pool, ws, s);
        if (verbose) {
            uint32_t top = 0;
            for (const SplitJob &l : pool.leaves) top = std::max(top, l.work);
            std::fprintf(stderr, "[peel] regrouped: %zu jobs (%lld edges, %lld wedges); %zu leaves (%lld edges, %lld wedges, up to %u in one) in all\n",
                         g.jobs.size(), (long long)g.m, (long long)g.n_w, pool.leaves.size(),
                         (long long)pool.m, (long long)pool.n_w, top);
        }
        jobs = g.jobs;
        if (!leaves && !pool.leaves.empty())
            leaves.reset(new LeafRun(pool, m, ix.n_w, phi_out, ask.unit, ng, turn,
                                     yield_word(turn), ws, s));
        if (jobs.empty()) break;
        // The compute units that the next sweep leaves peel the heaviest
        // leaves meanwhile: one of a few hundred thousand wedges takes tens of
        // milliseconds, all of them together little more.  5M-edge graph 262
        // and 247 ms, 192 pool graphs 151 and 142 ms.
        if (leaves && coop && g.m < kAllCusEdges) leaves->start(cus - peel_grid(tp, cus, cus));
        uint64_t *supl2 = ws.get<uint64_t>("sp_supl", g.m + 1);
        int64_t *loff2 = ws.get<int64_t>("sp_loff", g.m + 1);
        uint3 *link2 = ws.get<uint3>("sp_link", 2 * g.n_w + 1);
        regroup_links(g, supl2, loff2, link2, ws, s);
        cur.m = g.m;
        cur.n_b = g.n_b;
        cur.n_w = g.n_w;
        cur.bwoff = g.bwoff;
        cur.bk = g.bk;
        cur.wea = g.wea;
        cur.web = g.web;
        cur.wbl = g.wbl;
        cur.link_off = loff2;
        cur.link = link2;
        cur.oid = g.oid;
        ask.supl = supl2;
        ask.fixed = nullptr;
        ask.min_level = 0;
        ask.sup_out = nullptr;
    }
    if (leaves) leaves->finish(levels, max_level, pc);
    pc.launches += 1 + pc.yields;
    pc.max_phi = max_level;
    for (int32_t l : levels) pc.levels = std::max<int64_t>(pc.levels, l);
}

void peel_split(const RankCSR &r, IndexArrays &ix, const std::vector<int64_t> &off,
                int64_t *sup_out, int64_t *phi_out, PeelCounters &pc, Workspace &ws, hipStream_t s,
                const PeelOptions *opt) {
    const int32_t ng = (int32_t)off.size() - 1;
    const int64_t m = off[(size_t)ng];
    if (m == 0) return;
    const bool unit = opt && opt->unit_updates;
    const char *mv = std::getenv("BT_PEEL_MODE");
    const bool coop = ws.coop && !(mv && std::strcmp(mv, "graph") == 0);
    std::vector<SplitJob> jobs;
    for (int32_t g = 0; g < ng; ++g)
        if (off[(size_t)g + 1] > off[(size_t)g])
            jobs.push_back(SplitJob{0, (int32_t)off[(size_t)g],
                                    (int32_t)(off[(size_t)g + 1] - off[(size_t)g]), g, kLevelMax,
                                    (uint32_t)(ix.n_w * (off[(size_t)g + 1] - off[(size_t)g]) / m), false});
    std::unique_ptr<CoopTurn> turn;
    if (coop) turn.reset(new CoopTurn(m));
    const SplitIndex cur = view_of(ix, m);
    SweepAsk ask;
    ask.supl = ix.supl;
    ask.fixed = opt ? opt->fixed : nullptr;
    ask.min_level = opt ? opt->min_level : 0;
    ask.unit = unit;
    ask.least = opt && opt->plain;
    // Few levels: level by level as well, as splitting passes over the graph
    // once more.
    const bool few = opt && few_levels(std::min(ix.max_sup, opt->levels), ix.n_w);
    ask.plain = few || (opt && opt->plain);
    ask.sup_out = sup_out;
    ask.scratch = few ? nullptr : phi_out;
    if (ask.plain) return peel_levels(cur, jobs, ask, r.tp, turn.get(), phi_out, pc, ws, s);
    const PeelCounters before = pc;
    try {
        peel_parts(ix, cur, jobs, ask, ng, r.tp, coop, turn.get(), phi_out, pc, ws, s);
    } catch (const Error &e) {
        // What the split takes does not fit: level by level on the same index.
        if (e.status != BT_ENOMEM) throw;
        if (std::getenv("BT_PEEL_VERBOSE"))
            std::fprintf(stderr, "[peel] %s: level by level\n", e.msg.c_str());
        BT_HIP(hipStreamSynchronize(s));
        ws.drop(kSplitBuffers);
        rebuild_links(ix, m, s);
        pc = before;
        ask.plain = ask.least = true;
        peel_levels(cur, jobs, ask, r.tp, turn.get(), phi_out, pc, ws, s);
    }
}

}  // namespace bt
