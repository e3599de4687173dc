// peel_leaf.hip - the peel of small edge sets, one workgroup each.
//
// A graph of fewer than kLeafEdges edges (in a batch: each such graph) peels
// in one workgroup that keeps every edge's support, link range and state in
// LDS.  Its rounds are the bulk-synchronous rounds of Algorithm 5, as in the
// grid-wide peels, but what made those slow for small graphs is gone:
//   - a round ends in a workgroup barrier (about 0.1 us) instead of two grid
//     barriers (about 2.3 us each);
//   - supports fall by LDS atomics; the grid-wide peels issue each decrement
//     as a memory-side atomic (2.4e10/s for the whole chip);
//   - a wedge is alive exactly while neither of its edges has been removed,
//     which the edges' LDS states say, so there are no alive bits to clear.
// Graphs are independent, so a batch's graphs peel side by side on all CUs,
// pulled from a queue in decreasing size, and no graph waits for another's
// rounds.  A round still takes 4.7 to 6.6 us (graphs of 14,000 edges, 350 to
// 2,100 rounds; 9.4 us grid-wide): about 2 us in each phase, chains of work
// item, link, bloom state (a returning memory atomic) in phase A and work
// item, bloom state, wedge records in phase B, at 4 cycles an instruction.
// Counting the kills in an LDS hash table instead of memory did not shorten
// it, nor did the links' ends in LDS by more than 3%.  An edge that crosses
// the level waits in LDS for the end of its wave's phase, as queueing it takes
// another wait for memory, and phase B has four elements a lane in flight:
// 192 pool graphs' leaves 40 ms without either, 35 ms so.  512 graphs of 200 to
// 16,000 edges in one batch: 63.3 ms grid-wide, 18.8 ms so; the 10k-edge uniform
// graph 0.67 ms and 0.29 ms.
//
// The workgroup makes its own link lists (twin and bloom of each wedge of an
// edge) from the wedge records by counting in LDS, so the index build of
// these graphs stops at the wedges.
//
// Work items are pieces of at most 64 links (phase A) or wedges (phase B).
// Blooms of small graphs hold few wedges, so a wave takes up to 64 items at
// once and spreads their elements over its lanes: item j of a lane's element
// is found from a 64-bit mask of the items' first elements.
#include <algorithm>
#include <cstdlib>

#include "peel_split.h"

namespace bt {

namespace {

constexpr int kLeafBlock = 1024;
constexpr int kAhead = 4;   // elements per lane in flight in phase B
constexpr int kCross = 96;  // edges a wave holds back until they are queued (at least 64)
constexpr uint32_t kNoTwin = 0xffffffffu;  // the twin is not peeled here
// An edge's state: remaining, queued for an even or an odd round (1, 2), removed.
enum : uint8_t { kRemaining = 0, kRemoved = 3 };

// Jobs [j0, j1) of a list, handed out through `queue`.
struct LeafList {
    const LeafJob *jobs;
    const int32_t *order;  // jobs in queue order (null: as they are)
    int32_t *queue;
    int32_t j0, j1;
};

struct LeafArgs {
    LeafList list[kLeafLists];  // taken in turn
    int32_t n_lists;
    int32_t once;  // a workgroup takes one job
    // Nullable: the word that asks the launch to end early.  Workgroups from
    // `sure` on then take no job, and none takes another.
    const int32_t *yield;
    int32_t sure;
    const int32_t *wea, *web, *wbl;
    const uint32_t *bwoff;
    const int32_t *bk;  // initial bloom numbers
    u64 *bs;            // (live wedges at the round's start << 32) | kills this round
    uint2 *link;        // {bloom, twin}: job's links at [2 w0, 2 (w0 + nw))
    uint32_t *ends;     // end of each edge's links in its job's
    // Work lists past their part in LDS.
    uint2 *front[2];    // {edge | (links - 1) << 16, first link}
    uint2 *items;       // {bloom | multi << 31, first wedge << 6 | (wedges - 1)}; kLeafJobWedges
    const int32_t *oid;  // where an edge's number goes in phi_out (null: at the edge)
    int64_t *phi_out;
    int32_t *glevels;  // levels per graph
    LeafCtl *ctl;
};

// First slots of the job's regions of the work lists: an edge has at most
// one item more than its links / 64, a bloom one more than its wedges / 64.
__device__ __forceinline__ int64_t front_base(const LeafJob &J) {
    return (int64_t)J.e0 + J.w0 / 32 + J.id;
}
__device__ __forceinline__ int64_t items_base(const LeafJob &J) {
    return (int64_t)J.b0 + J.w0 / 64 + J.id;
}

// Each lane asks for cnt consecutive slots of a counter in LDS.  Must be
// called by all 64 lanes.
__device__ __forceinline__ uint32_t lds_alloc(uint32_t cnt, uint32_t *ctr) {
    const unsigned long long any = __ballot(cnt != 0);
    if (!any) return 0;
    uint32_t before, total;
    if (!__ballot(cnt > 1)) {
        before = (uint32_t)__popcll(any & lanemask_lt());
        total = (uint32_t)__popcll(any);
    } else {
        const uint32_t inc = wave_inclusive_sum<uint32_t>(cnt);
        total = wave_last(inc);
        before = inc - cnt;
    }
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(ctr, total);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + before;
}

// Writes a lane's n elements from lo as items of at most 64: {id | extra of
// the piece's size, position}.  A lane writes its first piece, the whole wave the
// others of a longer range.
template <typename F>
__device__ __forceinline__ void put_pieces(uint32_t n, uint32_t lo, uint32_t cnt, uint32_t slot,
                                           uint32_t id, F &&put) {
    if (cnt) put(slot, id, lo, min((uint32_t)kWave, n), cnt);
    unsigned long long big = __ballot(cnt > 1);
    while (big) {
        const int l = __ffsll(big) - 1;
        big &= big - 1;
        const uint32_t bn = __shfl(n, l, kWave), blo = __shfl(lo, l, kWave);
        const uint32_t bc = __shfl(cnt, l, kWave), bs = __shfl(slot, l, kWave);
        const uint32_t bi = __shfl(id, l, kWave);
        for (uint32_t c = 1 + lane_id(); c < bc; c += kWave)
            put(bs + c, bi, blo + c * kWave, min((uint32_t)kWave, bn - c * kWave), bc);
    }
}

// The lanes' items of elements t0 + lane, t0 + 64 + lane, ... (see item_of).
template <int U>
__device__ __forceinline__ void items_of(bool ok, uint32_t start, uint32_t t0, u64 *mask, int (&j)[U]) {
    int before = (int)__popcll(__ballot(ok && start < t0));
    if (lane_id() < U)
        __hip_atomic_store(&mask[lane_id()], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (ok && start >= t0 && start < t0 + U * kWave)
        __hip_atomic_fetch_or(&mask[(start - t0) / kWave], 1ull << ((start - t0) % kWave),
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const u64 le = lanemask_lt() | (u64(1) << lane_id());
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const u64 m = __hip_atomic_load(&mask[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        j[u] = before + (int)__popcll(m & le) - 1;
        before += (int)__popcll(m);
    }
}

// A bloom's state for the next round: its kills leave it.
__device__ __forceinline__ u64 settle(u64 state) {
    return (u64)((uint32_t)(state >> 32) - (uint32_t)state) << 32;
}

// A launch: jobs of up to ecap edges (a multiple of 4).  The work lists keep
// their first entries in LDS and the rest in global memory at the same index.
// Smaller jobs take less LDS and fewer waves, so that several share a compute
// unit.
struct LeafClass {
    int ecap, threads, front_lds, items_lds;
    // Frontier lists, bloom items; support and state of each edge.
    size_t lds() const { return sizeof(uint2) * (2 * front_lds + items_lds) + (size_t)ecap * 5; }
};
constexpr LeafClass kLeafClasses[] = {
    {(int)kLeafCap, 1024, 512, 1024}, {7168, 512, 256, 512}, {2048, 256, 128, 256}};
static_assert(sizeof kLeafClasses / sizeof *kLeafClasses == kNumLeafClasses, "a queue each");

int leaf_class(int64_t edges) {
    int c = 0;
    while (c + 1 < kNumLeafClasses && edges <= kLeafClasses[c + 1].ecap) ++c;
    return c;
}

template <bool UNIT>
__global__ __launch_bounds__(kLeafBlock) void k_peel_leaf(LeafArgs A, LeafClass K) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t front_lds = K.front_lds, items_lds = K.items_lds;
    uint2 *const lf0 = reinterpret_cast<uint2 *>(smem_raw), *const lf1 = lf0 + front_lds;
    uint2 *const li = lf1 + front_lds;
    int32_t *const sup = reinterpret_cast<int32_t *>(li + items_lds);
    uint8_t *const stt = reinterpret_cast<uint8_t *>(sup + K.ecap);
    __shared__ LeafJob s_job;
    __shared__ int32_t s_min[2];  // the next level, by the level's parity
    __shared__ uint32_t s_nf[2], s_ni[2], s_multi[2];
    __shared__ u64 s_mask[kLeafBlock / kWave][kAhead];
    __shared__ uint16_t s_cross[kLeafBlock / kWave][kCross];
    __shared__ uint32_t s_scan[kLeafBlock / kWave + 1];
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wv = tid / kWave, nwv = nthr / kWave;
    u64 *const mask = s_mask[wv];
    uint16_t *const cross = s_cross[wv];
    uint32_t upd = 0, unb = 0, touch = 0, visits = 0;  // of this lane
    u64 rounds = 0;  // thread 0's
    int32_t max_level = 0;
    int32_t list = 0;  // thread 0's
    bool done_one = false;

    for (bool more = true; more; more = !A.once, done_one = true) {
        __syncthreads();
        if (tid == 0) {
            s_job.ne = -1;
            const bool stop = A.yield && (done_one || (int32_t)blockIdx.x >= A.sure) &&
                              __hip_atomic_load(A.yield, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_SYSTEM) != 0;
            for (; !stop && list < A.n_lists; ++list) {
                const LeafList &L = A.list[list];
                const int32_t i = L.j0 + atomicAdd(L.queue, 1);
                if (i >= L.j1) continue;
                s_job = L.jobs[L.order ? L.order[i] : i];
                break;
            }
        }
        __syncthreads();
        const LeafJob J = s_job;
        if (J.ne < 0) break;
        const int32_t ne = J.ne, e0 = J.e0;
        if (ne <= 0 || ne > K.ecap) continue;  // the host queues none of these
        uint2 *const link = A.link + 2 * (int64_t)J.w0;
        uint2 *const fr0 = A.front[0] + front_base(J), *const fr1 = A.front[1] + front_base(J);
        uint2 *const items = A.items + items_base(J);

        // Links: counts (in LDS, where the supports go later), their prefix
        // sums, the links, and where each edge's end.
        uint32_t *const cur_end = reinterpret_cast<uint32_t *>(sup);
        uint32_t *const ends = A.ends + e0;
        for (int i = tid; i < ne; i += nthr) {
            cur_end[i] = 0;
            stt[i] = kRemaining;
        }
        // Edges past the end, up to a multiple of four, are removed ones.
        if (tid < 4 && ne + tid < ((ne + 3) & ~3)) stt[ne + tid] = kRemoved;
        if (tid == 0) {
            s_min[0] = INT_MAX;
            s_nf[0] = s_nf[1] = s_ni[0] = s_ni[1] = s_multi[0] = s_multi[1] = 0;
        }
        __syncthreads();
        for (uint32_t i = tid; i < J.nw; i += nthr) {
            const uint32_t a = (uint32_t)A.wea[J.w0 + i], b = (uint32_t)A.web[J.w0 + i];
            if (!(a & kFixedBit)) atomicAdd(&cur_end[a - e0], 1u);
            if (!(b & kFixedBit)) atomicAdd(&cur_end[b - e0], 1u);
        }
        __syncthreads();
        {
            // Each thread owns a run of edges.
            const int per = (ne + nthr - 1) / nthr;
            const int i0 = min(tid * per, ne), i1 = min(i0 + per, ne);
            uint32_t mine = 0;
            for (int i = i0; i < i1; ++i) mine += cur_end[i];
            uint32_t total;
            uint32_t run = block_exclusive_sum<uint32_t>(mine, s_scan, &total);
            for (int i = i0; i < i1; ++i) {
                const uint32_t c = cur_end[i];
                cur_end[i] = run;
                run += c;
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < J.nw; i += nthr) {
            const uint32_t w = J.w0 + i;
            const uint32_t bl = (uint32_t)A.wbl[w];
            const uint32_t a = (uint32_t)A.wea[w], b = (uint32_t)A.web[w];
            const uint32_t la = a & kFixedBit ? kNoTwin : a - (uint32_t)e0;
            const uint32_t lb = b & kFixedBit ? kNoTwin : b - (uint32_t)e0;
            if (la != kNoTwin) link[atomicAdd(&cur_end[la], 1u)] = make_uint2(bl, lb);
            if (lb != kNoTwin) link[atomicAdd(&cur_end[lb], 1u)] = make_uint2(bl, la);
        }
        __syncthreads();
        for (int i = tid; i < ne; i += nthr) {
            ends[i] = cur_end[i];
            sup[i] = 0;
        }
        __syncthreads();
        // Supports: a wedge of a k-bloom gives each of its edges k - 1
        // butterflies (Lemma 2).
        for (uint32_t i = tid; i < J.nw; i += nthr) {
            const uint32_t w = J.w0 + i;
            const int32_t d = A.bk[A.wbl[w]] - 1;
            if (d <= 0) continue;  // a part's spent bloom
            const uint32_t a = (uint32_t)A.wea[w], b = (uint32_t)A.web[w];
            if (!(a & kFixedBit)) atomicAdd(&sup[a - e0], d);
            if (!(b & kFixedBit)) atomicAdd(&sup[b - e0], d);
        }
        __syncthreads();

        // Queues edge t (lanes with pred) for the round of parity q; all 64
        // lanes call.  An edge without links needs no work item.
        const auto push_front = [&](bool pred, uint32_t t, int q, int32_t level) {
            if (!__ballot(pred)) return;
            uint32_t lo = 0, n = 0;
            if (pred) {
                A.phi_out[A.oid ? A.oid[e0 + t] : e0 + (int32_t)t] = level;
                stt[t] = (uint8_t)(1 + q);
                lo = t ? ends[t - 1] : 0u;
                n = ends[t] - lo;
            }
            if (!__ballot(n != 0)) return;
            const uint32_t cnt = (n + kWave - 1) / kWave;
            const uint32_t slot = lds_alloc(cnt, &s_nf[q]);
            uint2 *const list = q ? fr1 : fr0, *const near = q ? lf1 : lf0;
            put_pieces(n, lo, cnt, slot, t,
                       [&](uint32_t s, uint32_t id, uint32_t at, uint32_t len, uint32_t) {
                           const uint2 v = make_uint2(id | ((len - 1) << 16), at);
                           if (s < front_lds) near[s] = v;
                           else list[s] = v;
                       });
        };

        // An edge that crosses the level is noted (in LDS) and queued with
        // others at the end of its wave's phase: queueing waits for memory.
        uint32_t n_cross = 0;
        const auto queue_crossed = [&](int q, int32_t level) {
            for (uint32_t i = 0; i < n_cross; i += kWave) {
                const bool has = i + lane_id() < n_cross;
                push_front(has, has ? cross[i + lane_id()] : 0u, q, level);
            }
            n_cross = 0;
        };
        const auto crossed = [&](bool pred, uint32_t t, int q, int32_t level) {
            const u64 who = __ballot(pred);
            if (!who) return;
            const uint32_t n = (uint32_t)__popcll(who);
            if (n_cross + n > kCross) queue_crossed(q, level);
            if (pred) cross[n_cross + (uint32_t)__popcll(who & lanemask_lt())] = (uint16_t)t;
            n_cross += n;
        };

        int32_t levels = 0;
        int r = 0;
        while (true) {
            // The next level: the smallest support among the remaining edges
            // (INT_MAX for the others), four edges a thread and step.
            const auto remaining = [&](int i) {
                uint32_t s4 = ~0u;
                int4 x = make_int4(0, 0, 0, 0);
                if (i < ne) {
                    s4 = *reinterpret_cast<const uint32_t *>(&stt[i]);
                    x = *reinterpret_cast<const int4 *>(&sup[i]);
                }
                return make_int4(s4 & 0xffu ? INT_MAX : x.x, s4 & 0xff00u ? INT_MAX : x.y,
                                 s4 & 0xff0000u ? INT_MAX : x.z, s4 & 0xff000000u ? INT_MAX : x.w);
            };
            int32_t mn = INT_MAX;
            for (int i = 4 * tid; i < ne; i += 4 * nthr) {
                const int4 v = remaining(i);
                mn = min(mn, min(min(v.x, v.y), min(v.z, v.w)));
            }
            mn = wave_min(mn);
            // The other word is cleared for the level after this one.  It was
            // last read before the barrier that ended the last level's queueing,
            // and is next lowered after the one below: a level whose edges have
            // no links runs no round, so no barrier but these two lies between
            // one level's minimum and the next one's.
            if (tid == 0) s_min[(levels & 1) ^ 1] = INT_MAX;
            if (lane_id() == 0 && mn != INT_MAX) atomicMin(&s_min[levels & 1], mn);
            __syncthreads();
            const int32_t level = s_min[levels & 1];
            if (level == INT_MAX) break;
            if (mn == level) {  // only waves that hold such an edge look again
                for (int i0 = 0; i0 < ne; i0 += 4 * nthr) {
                    const int i = i0 + 4 * tid;
                    const int4 v = remaining(i);
                    push_front(v.x == level, (uint32_t)i, r & 1, level);
                    push_front(v.y == level, (uint32_t)i + 1, r & 1, level);
                    push_front(v.z == level, (uint32_t)i + 2, r & 1, level);
                    push_front(v.w == level, (uint32_t)i + 3, r & 1, level);
                }
            }
            __syncthreads();
            ++levels;
            if (level > max_level) max_level = level;
            uint32_t nf = s_nf[r & 1];
            while (nf > 0) {
                const int p = r & 1, q = p ^ 1;
                const uint8_t cur = (uint8_t)(1 + p), nxt = (uint8_t)(1 + q);
                const uint2 *const fl = p ? fr1 : fr0, *const fn = p ? lf1 : lf0;
                const auto front_item = [&](uint32_t i) { return i < front_lds ? fn[i] : fl[i]; };
                // Phase A: the frontier's links.  A wedge whose edges are both
                // in the frontier is killed by the smaller one.
                {
                    const uint32_t per = min((uint32_t)kWave, (nf + nwv - 1) / nwv);
                    for (uint32_t g0 = wv * per; g0 < nf; g0 += nwv * per) {
                        const bool ok = (uint32_t)lane_id() < per && g0 + lane_id() < nf;
                        uint2 it = make_uint2(0, 0);
                        if (ok) it = front_item(g0 + lane_id());
                        const uint32_t n = ok ? (it.x >> 16) + 1 : 0u;
                        const uint32_t e = it.x & 0xffffu;
                        const uint32_t inc = wave_inclusive_sum<uint32_t>(n);
                        const uint32_t start = inc - n;
                        const uint32_t total = wave_last(inc);
                        for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
                            const int j = item_of(ok, start, t0, mask);
                            const uint32_t x = t0 + lane_id();
                            const bool act = x < total;
                            const uint32_t ej = __shfl(e, j, kWave);
                            const uint32_t at = __shfl(it.y - start, j, kWave) + x;
                            uint32_t bl = 0, t = kNoTwin, w0 = 0, w1 = 0;
                            uint8_t s = kRemaining;
                            u64 old = 1;
                            bool alive = false;
                            if (act) {
                                const uint2 lk = link[at];
                                bl = lk.x;
                                t = lk.y;
                                if (t != kNoTwin) s = stt[t];
                                alive = s != kRemoved && !(s == cur && t < ej);
                                w0 = A.bwoff[bl];
                                w1 = A.bwoff[bl + 1];
                                if (alive) old = atomicAdd(&A.bs[bl], (u64)1);
                            }
                            // The twin, if it stays, loses its k - 1 butterflies.
                            const int32_t kb = (int32_t)(old >> 32), d = kb - 1;
                            const bool dec = alive && t != kNoTwin && s != cur && d > 0;
                            int32_t o = 0;
                            if (dec) o = atomicSub(&sup[t], d);
                            crossed(dec && o > level && o - d <= level, t, q, level);
                            upd += dec ? 1 : 0;
                            // The bloom's first kill this round queues it.
                            const bool first = alive && (uint32_t)old == 0 && kb > 1;
                            if (__ballot(first)) {
                                const uint32_t len = first ? w1 - w0 : 0u;
                                const uint32_t cnt = (len + kWave - 1) / kWave;
                                const uint32_t slot = lds_alloc(cnt, &s_ni[p]);
                                if (cnt > 1) s_multi[p] = 1;
                                put_pieces(len, w0 - J.w0, cnt, slot, bl,
                                           [&](uint32_t sl, uint32_t id, uint32_t pos, uint32_t pn,
                                               uint32_t pieces) {
                                               const uint2 v = make_uint2(
                                                   id | (pieces > 1 ? 0x80000000u : 0u),
                                                   (pos << 6) | (pn - 1));
                                               if (sl < items_lds) li[sl] = v;
                                               else items[sl] = v;
                                           });
                            }
                        }
                    }
                    queue_crossed(q, level);
                }
                __syncthreads();
                const uint32_t ni = s_ni[p];
                const bool multi = s_multi[p] != 0;
                if (tid == 0) {
                    s_nf[p] = 0;
                    s_ni[q] = 0;
                    s_multi[q] = 0;
                    rounds += 1;
                }
                for (uint32_t i = tid; i < nf; i += nthr) stt[front_item(i).x & 0xffffu] = kRemoved;
                // Phase B: survivors of touched blooms lose their C kills.
                {
                    const uint32_t per = min((uint32_t)kWave, (ni + nwv - 1) / nwv);
                    for (uint32_t g0 = wv * per; g0 < ni; g0 += nwv * per) {
                        const uint32_t i = g0 + lane_id();
                        const bool ok = (uint32_t)lane_id() < per && i < ni;
                        uint2 it = make_uint2(0, 0);
                        u64 state = 0;
                        if (ok) {
                            it = i < items_lds ? li[i] : items[i];
                            state = ld(&A.bs[it.x & kEdgeMask]);  // arrives with the wedges
                        }
                        const uint32_t n = ok ? (it.y & 63u) + 1 : 0u;
                        const uint32_t inc = wave_inclusive_sum<uint32_t>(n);
                        const uint32_t start = inc - n;
                        const uint32_t total = wave_last(inc);
                        for (uint32_t t0 = 0; t0 < total; t0 += kAhead * kWave) {
                            int j[kAhead];
                            uint32_t a[kAhead], b[kAhead];
                            items_of(ok, start, t0, mask, j);
#pragma unroll
                            for (int u = 0; u < kAhead; ++u) {
                                const uint32_t x = t0 + u * kWave + lane_id();
                                a[u] = b[u] = kFixedBit;
                                if (t0 + u * kWave >= total) continue;
                                const uint32_t w =
                                    J.w0 + __shfl((it.y >> 6) - start, j[u], kWave) + x;
                                if (x < total) {
                                    a[u] = (uint32_t)A.wea[w];
                                    b[u] = (uint32_t)A.web[w];
                                }
                            }
#pragma unroll
                            for (int u = 0; u < kAhead; ++u) {
                                if (t0 + u * kWave >= total) break;
                                const bool act = t0 + u * kWave + lane_id() < total;
                                const int32_t cj = __shfl((int32_t)(uint32_t)state, j[u], kWave);
                                const bool oa = !(a[u] & kFixedBit), ob = !(b[u] & kFixedBit);
                                const uint32_t la = a[u] - (uint32_t)e0, lb = b[u] - (uint32_t)e0;
                                const uint8_t sa = oa ? stt[la] : (uint8_t)kRemaining;
                                const uint8_t sb = ob ? stt[lb] : (uint8_t)kRemaining;
                                const bool live = act && (sa == kRemaining || sa == nxt) &&
                                                  (sb == kRemaining || sb == nxt);
                                const bool da = live && oa, db = live && ob;
                                bool f1 = false, f2 = false;
                                if (UNIT) {
                                    // Without batch bloom processing: one unit per
                                    // kill; the step from level + 1 crosses.
                                    for (int32_t c = 0; c < (live ? cj : 0); ++c) {
                                        if (da) f1 |= atomicSub(&sup[la], 1) == level + 1;
                                        if (db) f2 |= atomicSub(&sup[lb], 1) == level + 1;
                                    }
                                    upd += (uint32_t)((da ? cj : 0) + (db ? cj : 0));
                                } else {
                                    int32_t o1 = 0, o2 = 0;
                                    if (da) o1 = atomicSub(&sup[la], cj);
                                    if (db) o2 = atomicSub(&sup[lb], cj);
                                    f1 = da && o1 > level && o1 - cj <= level;
                                    f2 = db && o2 > level && o2 - cj <= level;
                                    upd += (da ? 1u : 0u) + (db ? 1u : 0u);
                                    unb += (uint32_t)((da ? cj - 1 : 0) + (db ? cj - 1 : 0));
                                }
                                touch += live ? 1 : 0;
                                crossed(f1, la, q, level);
                                crossed(f2, lb, q, level);
                            }
                        }
                        // A bloom of one piece is settled by its reader.
                        if (ok && !(it.x & 0x80000000u)) {
                            st(&A.bs[it.x], settle(state));
                            visits += 1;
                        }
                    }
                    queue_crossed(q, level);
                }
                __syncthreads();
                if (multi) {
                    for (uint32_t i = tid; i < ni; i += nthr) {
                        const uint2 it = i < items_lds ? li[i] : items[i];
                        const uint32_t b = it.x & kEdgeMask;
                        if (!(it.x & 0x80000000u) || A.bwoff[b] != J.w0 + (it.y >> 6)) continue;
                        st(&A.bs[b], settle(ld(&A.bs[b])));
                        visits += 1;
                    }
                    __syncthreads();
                }
                ++r;
                nf = s_nf[r & 1];
            }
        }
        if (tid == 0) atomicAdd(&A.glevels[J.graph], levels);
    }
    const u64 uu = wave_sum<u64>(upd), bb = wave_sum<u64>(unb), tt = wave_sum<u64>(touch),
              vv = wave_sum<u64>(visits);
    if (lane_id() == 0) {
        if (uu) atomicAdd(&A.ctl->updates, uu);
        if (bb) atomicAdd(&A.ctl->unbatched, bb);
        if (tt) atomicAdd(&A.ctl->touched, tt);
        if (vv) atomicAdd(&A.ctl->bloom_visits, vv);
    }
    if (tid == 0) {
        if (rounds) atomicAdd(&A.ctl->rounds, rounds);
        atomicMax(&A.ctl->max_level, max_level);
    }
}

// The jobs of a union's small graphs: graph g's edges [off[g], off[g + 1]),
// its blooms and wedges from its bases to where its cursor stopped.
__global__ void k_leaf_jobs(const int64_t *off, int32_t ng, const uint64_t *base,
                            const uint64_t *cursor, LeafJob *jobs, LeafCtl *ctl) {
    u64 nb = 0, nw = 0;
    for (int32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < ng; g += gridDim.x * blockDim.x) {
        LeafJob J;
        J.e0 = (int32_t)off[g];
        J.ne = (int32_t)(off[g + 1] - off[g]);
        J.w0 = (uint32_t)base[g];
        J.nw = (uint32_t)cursor[g] - J.w0;
        J.b0 = (uint32_t)(base[g] >> 32);
        J.nb = (uint32_t)(cursor[g] >> 32) - J.b0;
        J.graph = g;
        J.id = g;
        jobs[g] = J;
        nb += J.nb;
        nw += J.nw;
    }
    nb = wave_sum(nb);
    nw = wave_sum(nw);
    if (lane_id() == 0) {
        if (nb) atomicAdd(&ctl->blooms, nb);
        if (nw) atomicAdd(&ctl->wedges, nw);
    }
}

// Bloom states; slots between the graphs' regions hold leftovers, unused.
__global__ void k_leaf_state(const int32_t *bk, int64_t n, u64 *bs) {
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < n;
         b += (int64_t)gridDim.x * blockDim.x)
        bs[b] = (u64)(uint32_t)bk[b] << 32;
}

}  // namespace

int64_t peel_leaf_bytes(int64_t m, int64_t cap_b, int64_t cap_w, int64_t graphs) {
    const int64_t front = m + cap_w / 32 + graphs + 1, items = cap_b + cap_w / 64 + graphs + 1;
    const int64_t t = 16 * cap_w + 4 * m + 16 * front + 8 * items + 8 * (cap_b + 1) + 48 * graphs + 4096;
    return t + t / 8;
}

namespace {

// Buffers of a leaf peel over arrays of m edges, n_b blooms and n_w wedges.
LeafArgs leaf_args(int64_t m, int64_t n_b, int64_t n_w, int64_t n_jobs, int32_t n_roots,
                   Workspace &ws, hipStream_t s) {
    LeafArgs A{};
    A.bs = ws.get<u64>("lf_bs", n_b + 1);
    A.link = ws.get<uint2>("lf_link", 2 * n_w + 1);
    A.ends = ws.get<uint32_t>("lf_ends", m);
    A.front[0] = ws.get<uint2>("lf_front0", m + n_w / 32 + n_jobs + 1);
    A.front[1] = ws.get<uint2>("lf_front1", m + n_w / 32 + n_jobs + 1);
    A.items = ws.get<uint2>("lf_items", n_b + n_w / 64 + n_jobs + 1);
    A.glevels = ws.get<int32_t>("lf_levels", n_roots);
    A.ctl = ws.get<LeafCtl>("lf_ctl", 1);
    zero_bytes(A.ctl, sizeof(LeafCtl), s);
    zero_bytes(A.glevels, sizeof(int32_t) * n_roots, s);
    return A;
}

void leaf_state(const LeafArgs &A, int64_t b0, int64_t n, hipStream_t s) {
    k_leaf_state<<<grid_for(n, 256, 8192), 256, 0, s>>>(A.bk + b0, n, A.bs + b0);
    BT_CHECK_LAUNCH();
}

// Workgroups of a launch that take a job whatever the yield word says, so that
// a launch between two yields gets on; the other CUs are free for who asked.
constexpr int kSureLeaves = 64;

// Launches class c over A's lists, in which n jobs are left, by at most `most`
// workgroups.
void launch_leaves(LeafArgs A, int c, int64_t n, bool unit_updates, int most, hipStream_t s) {
    const auto kern = unit_updates ? k_peel_leaf<true> : k_peel_leaf<false>;
    const LeafClass &K = kLeafClasses[c];
    BT_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kLeafClasses[0].lds()));
    // Without a limit each job has a workgroup: one that took job after job
    // would hold its CU, and small requests' peels on other streams would wait
    // for the last of a large graph's leaves (small requests served beside
    // 2M-edge graphs: 30 ms in the middle, 12 to 28 ms so, and 2.1 to 2.5 ms
    // since those leaves that have not begun make room for them).
    const int64_t grid = std::min<int64_t>(n, most);
    A.once = grid == n ? 1 : 0;
    A.sure = kSureLeaves;
    if (grid <= 0) return;
    kern<<<(unsigned)grid, K.threads, K.lds(), s>>>(A, K);
    BT_CHECK_LAUNCH();
}

// Runs lists of jobs (lists[l][c]: list l's jobs of class c) to their end and
// reads the counters back.  `early` (nullable): the end of a launch that has
// taken from them already.  `turn` (nullable): held, with A.yield its word.
void run_leaves(LeafArgs A, const std::vector<std::vector<LeafList>> &lists, hipEvent_t early,
                bool unit_updates, int32_t n_roots, std::vector<int32_t> &levels, int32_t &max_level, PeelCounters &pc,
                LeafCtl &done, CoopTurn *turn, Workspace &ws, hipStream_t s) {
    hipEvent_t ev0, ev1;
    BT_HIP(hipEventCreate(&ev0));
    BT_HIP(hipEventCreate(&ev1));
    // The classes run beside each other on side streams (one after another
    // they took the sum of their longest jobs: 24 ms against 14 for 512 graphs
    // of up to 16,000 edges).
    hipEvent_t joins[kNumLeafClasses] = {};
    struct EvFree {
        hipEvent_t a, b, *e;
        Workspace &ws;
        bool joined;  // nothing runs on a side stream that s does not wait for
        ~EvFree() {
            if (!joined) ws.sync_sides();
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
            for (int c = 0; c < kNumLeafClasses; ++c)
                if (e[c]) (void)hipEventDestroy(e[c]);
        }
    } ev_free{ev0, ev1, joins, ws, true};
    LeafCtl *hc =
        reinterpret_cast<LeafCtl *>(ws.host((int)(sizeof(LeafCtl) / 8 + 1 + (n_roots + 1) / 2)));
    int32_t *hl = reinterpret_cast<int32_t *>(hc + 1);
    // Jobs of class c that no workgroup has taken.
    const auto left = [&](int c, bool begun) {
        int64_t n = 0;
        for (const auto &L : lists) {
            const LeafList &l = L[(size_t)c];
            const int32_t taken = begun ? hc->queue[&L - lists.data()][c] : 0;
            n += std::max(l.j1 - l.j0 - taken, 0);
        }
        return n;
    };
    float ms = 0.f;
    int64_t n_jobs = 0;
    for (bool begun = false;; begun = true) {
        int64_t n[kNumLeafClasses], all = 0;
        int last = -1;
        for (int c = 0; c < kNumLeafClasses; ++c) {
            all += n[c] = left(c, begun);
            if (n[c]) last = c;
        }
        if (begun) {
            if (all == 0) break;
            if (!turn) throw Error{BT_EDEVICE, "leaves were left over"};
            pc.yields += 1;
            turn->requeue();
        } else {
            n_jobs = all;
        }
        BT_HIP(hipEventRecord(ev0, s));
        ev_free.joined = false;
        for (int c = 0; c < kNumLeafClasses; ++c) {
            if (!n[c]) continue;
            A.n_lists = 0;
            for (const auto &l : lists)
                if (l[(size_t)c].j1 > l[(size_t)c].j0) A.list[A.n_lists++] = l[(size_t)c];
            const hipStream_t cs = c == last ? s : ws.side(c);  // the last class stays on s
            if (cs != s) BT_HIP(hipStreamWaitEvent(cs, ev0, 0));
            launch_leaves(A, c, n[c], unit_updates, INT_MAX, cs);
            if (cs != s) {
                if (!joins[c]) BT_HIP(hipEventCreateWithFlags(&joins[c], hipEventDisableTiming));
                BT_HIP(hipEventRecord(joins[c], cs));
            }
        }
        for (int c = 0; c < kNumLeafClasses; ++c)
            if (n[c] && c != last) BT_HIP(hipStreamWaitEvent(s, joins[c], 0));
        ev_free.joined = true;
        if (early && !begun) BT_HIP(hipStreamWaitEvent(s, early, 0));
        BT_HIP(hipEventRecord(ev1, s));
        BT_HIP(hipMemcpyAsync(hc, A.ctl, sizeof(LeafCtl), hipMemcpyDeviceToHost, s));
        BT_HIP(hipStreamSynchronize(s));
        float t = 0.f;
        BT_HIP(hipEventElapsedTime(&t, ev0, ev1));
        ms += t;
    }
    BT_HIP(hipMemcpyAsync(hl, A.glevels, sizeof(int32_t) * n_roots, hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    if (std::getenv("BT_PEEL_VERBOSE"))
        std::fprintf(stderr, "[peel] leaves: %lld: %.2f ms, %llu rounds\n", (long long)n_jobs,
                     (double)ms, hc->rounds);
    pc.kernel_ms += ms;
    pc.rounds += (int64_t)hc->rounds;
    pc.updates += (int64_t)hc->updates;
    pc.updates_unbatched += (int64_t)(hc->updates + hc->unbatched);
    pc.bloom_visits += (int64_t)hc->bloom_visits;
    pc.touched += (int64_t)hc->touched;
    max_level = std::max(max_level, hc->max_level);
    for (int32_t g = 0; g < n_roots; ++g) levels[(size_t)g] += hl[g];
    done = *hc;
}

}  // namespace

void peel_leaf(IndexArrays &ix, const std::vector<int64_t> &off, const int64_t *doff,
               int64_t *sup_out, int64_t *phi_out, bool unit_updates, PeelCounters &pc,
               Workspace &ws, hipStream_t s) {
    const int32_t ng = (int32_t)off.size() - 1;
    const int64_t m = off[(size_t)ng];
    if (m == 0) return;
    LeafArgs A = leaf_args(m, ix.cap_b, ix.cap_w, ng, ng, ws, s);
    LeafJob *jobs = ws.get<LeafJob>("lf_jobs", ng);
    A.bk = ix.bk;
    leaf_state(A, 0, ix.cap_b + 1, s);
    A.wea = ix.wea;
    A.web = ix.web;
    A.wbl = ix.wbl;
    A.bwoff = ix.bwoff;
    A.phi_out = phi_out;
    k_leaf_jobs<<<grid_for(ng, 256, 256), 256, 0, s>>>(doff, ng, ix.base, ix.cursor, jobs, A.ctl);
    BT_CHECK_LAUNCH();
    if (sup_out) supl_to_sup(ix.supl, sup_out, m, s);
    // This peel needs no co-resident workgroups, so it begins at once, beside
    // another that holds the turn; one of a much larger graph gives way.
    CoopTurn turn(m, false);
    std::vector<int32_t> levels((size_t)ng, 0);
    int32_t max_level = 0;
    LeafCtl done;
    // The graphs come in decreasing size, so by class.
    std::vector<std::vector<LeafList>> lists(1);
    for (int32_t c = 0, a = 0; c < kNumLeafClasses; ++c) {
        int32_t b = a;
        while (b < ng && leaf_class(off[(size_t)b + 1] - off[(size_t)b]) == c) ++b;
        lists[0].push_back(LeafList{jobs, nullptr, &A.ctl->queue[0][c], a, b});
        a = b;
    }
    run_leaves(A, lists, nullptr, unit_updates, ng, levels, max_level, pc, done, nullptr, ws, s);
    pc.launches += 1;
    pc.max_phi = max_level;
    for (int32_t l : levels) pc.levels = std::max<int64_t>(pc.levels, l);
    ix.n_b = (int64_t)done.blooms;
    ix.n_w = (int64_t)done.wedges;
}

// State of a pool's leaves while they are run in lists.
struct LeafRun::State {
    LeafArgs A;
    std::vector<std::vector<LeafList>> lists;
    size_t taken = 0;       // leaves in lists
    int64_t b_taken = 0;    // blooms of theirs
    hipEvent_t early = nullptr;  // the end of an early launch
    hipStream_t stream = nullptr;
};

LeafRun::LeafRun(const LeafPool &pool, int64_t m, int64_t n_w, int64_t *phi_out, bool unit_updates,
                 int32_t n_roots, CoopTurn *turn, const int32_t *yield_word, Workspace &ws,
                 hipStream_t s)
    : pool_(pool), unit_(unit_updates), roots_(n_roots), turn_(turn), ws_(ws), s_(s), st_(new State()) {
    LeafArgs &A = st_->A;
    // A leaf holds an edge or more, a bloom a wedge or more; a depth's blooms
    // have a slot more than there are.
    A = leaf_args(m, n_w + 64, n_w, m, n_roots, ws, s);
    A.bk = pool.bk;
    A.wea = pool.wea;
    A.web = pool.web;
    A.wbl = pool.wbl;
    A.bwoff = pool.bwoff;
    A.oid = pool.oid;
    A.phi_out = phi_out;
    A.yield = yield_word;
}

LeafRun::~LeafRun() {
    if (st_->early) {
        (void)hipStreamSynchronize(st_->stream);  // its buffers go with the workspace
        (void)hipEventDestroy(st_->early);
    }
}

// The leaves that are in no list yet, as a list: by class, then the heaviest first.
void LeafRun::take() {
    State &S = *st_;
    const int l = (int)S.lists.size();
    const size_t n = pool_.leaves.size() - S.taken;
    std::vector<int32_t> order(n);
    for (size_t j = 0; j < n; ++j) order[j] = (int32_t)j;
    const auto leaf = [&](int32_t j) -> const SplitJob & { return pool_.leaves[S.taken + (size_t)j]; };
    for (size_t j = S.taken; j < pool_.jobs.size(); ++j)
        if (pool_.jobs[j].nw >= kLeafJobWedges)
            throw Error{BT_EDEVICE, "a leaf holds more wedges than its work items can name"};
    std::sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        const int cx = leaf_class(leaf(x).ne), cy = leaf_class(leaf(y).ne);
        if (cx != cy) return cx < cy;
        return leaf(x).work != leaf(y).work ? leaf(x).work > leaf(y).work : x < y;
    });
    const char *const names[kLeafLists][2] = {
        {"lf_jobs", "lf_order"}, {"lf_jobs1", "lf_order1"}, {"lf_jobs2", "lf_order2"}};
    LeafJob *jobs = ws_.get<LeafJob>(names[l][0], (int64_t)n);
    int32_t *dorder = ws_.get<int32_t>(names[l][1], (int64_t)n);
    BT_HIP(hipMemcpyAsync(jobs, pool_.jobs.data() + S.taken, sizeof(LeafJob) * n,
                          hipMemcpyHostToDevice, s_));
    BT_HIP(hipMemcpyAsync(dorder, order.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s_));
    BT_HIP(hipStreamSynchronize(s_));  // the host arrays are read until here
    if (pool_.n_b > S.b_taken) leaf_state(S.A, S.b_taken, pool_.n_b - S.b_taken, s_);
    std::vector<LeafList> list;
    for (int32_t c = 0, a = 0; c < kNumLeafClasses; ++c) {
        int32_t b = a;
        while (b < (int32_t)n && leaf_class(leaf(order[(size_t)b]).ne) == c) ++b;
        list.push_back(LeafList{jobs, dorder, &S.A.ctl->queue[l][c], a, b});
        a = b;
    }
    S.lists.push_back(std::move(list));
    S.taken = pool_.leaves.size();
    S.b_taken = pool_.n_b;
}

void LeafRun::start(int groups) {
    State &S = *st_;
    if (pool_.leaves.size() == S.taken || groups <= 0 || (int)S.lists.size() + 1 >= kLeafLists) return;
    if (S.early) {
        if (hipEventQuery(S.early) != hipSuccess) {  // the last ones still run
            (void)hipGetLastError();
            return;
        }
    } else {
        BT_HIP(hipEventCreateWithFlags(&S.early, hipEventDisableTiming));
        S.stream = ws_.side(2);  // the others run classes at the end
    }
    take();
    hipEvent_t ready;
    BT_HIP(hipEventCreateWithFlags(&ready, hipEventDisableTiming));
    BT_HIP(hipEventRecord(ready, s_));
    BT_HIP(hipStreamWaitEvent(S.stream, ready, 0));
    BT_HIP(hipEventDestroy(ready));
    LeafArgs A = S.A;
    A.n_lists = 1;
    A.list[0] = S.lists.back()[0];
    launch_leaves(A, 0, A.list[0].j1 - A.list[0].j0, unit_, groups, S.stream);
    BT_HIP(hipEventRecord(S.early, S.stream));
}

void LeafRun::finish(std::vector<int32_t> &levels, int32_t &max_level, PeelCounters &pc) {
    State &S = *st_;
    if (pool_.leaves.size() > S.taken) take();
    if (S.lists.empty()) return;
    LeafCtl done;
    run_leaves(S.A, S.lists, S.early, unit_, roots_, levels, max_level, pc, done, turn_, ws_, s_);
}

}  // namespace bt
