// peel_common.h - device helpers of the peels: coherent loads and stores of
// shared state, wave-level slot allocation, the two-level grid barrier; the
// turns that peels take on the device.
#pragma once

#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "pipeline.h"

namespace bt {

// Cooperative peel kernels hold every CU until their last round; two of
// them at once (from different threads or engine slots) could each wait at
// a grid barrier for blocks the other keeps from being scheduled.  They
// therefore take turns in the process, in the order they asked.  While a
// turn is held, a waiter that weighs under 1/8 of the holder raises the
// holder's yield word (pinned host memory that its kernels read); a sweep then
// ends its launch between two rounds, a launch of leaves when the leaves begun
// are done, and the host thread queues again and relaunches from the state
// left in device memory.
class CoopTurn {
  public:
    // Blocks until this turn comes.  The turn weighs `weight` (the peel's
    // edges) unless the calling thread set another weight for its turns.
    // With barriers false the peel launches no cooperative kernel: it goes
    // beside the holder at once, which it makes yield as a waiter does.
    explicit CoopTurn(int64_t weight, bool barriers = true);
    ~CoopTurn();
    CoopTurn(const CoopTurn &) = delete;
    CoopTurn &operator=(const CoopTurn &) = delete;
    // Device address of the yield word (nonzero: a lighter peel waits).
    // With force, a word that always reads 1, for tests of the resume path.
    const int32_t *yield_word(bool force) const;
    // Gives the device up, queues behind every current waiter and returns
    // when the turn comes again and the much lighter peels that went beside
    // have ended.
    void requeue();

  private:
    uint64_t ticket_ = 0;
    int64_t weight_ = 0;
    bool held_ = true;  // false: beside the holder
};

namespace {

constexpr int kLinkChunk = kWave;   // links per phase-A work item (one per lane)
// Progressive mode: edge ids in wedge records and link twins carry this bit
// when the edge's bitruss number was fixed in an earlier pass; such edges
// keep their blooms alive but are never decremented or removed.
constexpr uint32_t kFixedBit = 0x80000000u;
constexpr uint32_t kEdgeMask = 0x7fffffffu;
constexpr int kWedgeChunk = kWave;  // wedges per phase-B work item (one per lane)
typedef unsigned long long u64;

// A counter alone on its cache line (contended atomics do not share lines).
struct alignas(128) Counter {
    u64 v;
};

struct alignas(16) FrontItem {
    int32_t e;        // < 0: none
    int32_t part;
    uint32_t lo, hi;  // link positions of this chunk
};

// Coherent access to state that blocks share within one launch.  The eight
// XCDs keep separate L2 caches; device-scope loads and stores (relaxed
// atomics) go to the point of coherence, so no round needs the L2 write-back
// and invalidation that a device-scope fence costs, and the read-only index
// stays cached in L2 across rounds.  Every access to mutable peel state
// inside a launch goes through these.
template <typename T> __device__ __forceinline__ T ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 16-byte work items move as two coherent 8-byte halves.
template <typename Item> __device__ __forceinline__ void st_item(Item *p, const Item &v) {
    static_assert(sizeof(Item) == 16, "work items are 16 bytes");
    u64 h[2];
    __builtin_memcpy(h, &v, 16);
    st(reinterpret_cast<u64 *>(p), h[0]);
    st(reinterpret_cast<u64 *>(p) + 1, h[1]);
}
template <typename Item> __device__ __forceinline__ Item ld_item(const Item *p) {
    u64 h[2];
    h[0] = ld(reinterpret_cast<const u64 *>(p));
    h[1] = ld(reinterpret_cast<const u64 *>(p) + 1);
    Item v;
    __builtin_memcpy(&v, h, 16);
    return v;
}

// Each lane asks for `cnt` consecutive slots of *counter; one atomic per
// wave.  Must be called by all 64 lanes.
__device__ __forceinline__ u64 wave_alloc(uint32_t cnt, u64 *counter) {
    const u64 inc = wave_inclusive_sum<u64>((u64)cnt);
    const u64 total = __shfl(inc, kWave - 1, kWave);
    u64 base = 0;
    if (lane_id() == kWave - 1 && total) base = atomicAdd(counter, total);
    base = __shfl(base, kWave - 1, kWave);
    return base + inc - cnt;
}

// Slot requests against up to three counters (a null counter takes no
// requests): each wave issues its atomics together and waits once.  Must be
// called by all 64 lanes.
__device__ __forceinline__ void wave_alloc3(uint32_t c0, u64 *k0, uint32_t c1, u64 *k1,
                                            uint32_t c2, u64 *k2, u64 (&base)[3]) {
    const uint32_t cnt[3] = {c0, c1, c2};
    u64 *const ctr[3] = {k0, k1, k2};
    uint32_t inc[3], tot[3];  // a wave's requests stay far below 2^32
    u64 r[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        inc[k] = wave_inclusive_sum<uint32_t>(cnt[k]);
        tot[k] = __shfl(inc[k], kWave - 1, kWave);
    }
    if (lane_id() == kWave - 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (tot[k]) r[k] = atomicAdd(ctr[k], (u64)tot[k]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) base[k] = __shfl(r[k], kWave - 1, kWave) + (inc[k] - cnt[k]);
}

// The item of element t0 + lane when the lanes' items start at `start`
// (increasing over the lanes with ok): the items that start before the
// window, plus those that start in it at or before this element, less one.
__device__ __forceinline__ int item_of(bool ok, uint32_t start, uint32_t t0, u64 *mask) {
    const int before = (int)__popcll(__ballot(ok && start < t0));
    if (lane_id() == 0) __hip_atomic_store(mask, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (ok && start >= t0 && start < t0 + kWave)
        __hip_atomic_fetch_or(mask, 1ull << (start - t0), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_WORKGROUP);
    const u64 m = __hip_atomic_load(mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const u64 le = lanemask_lt() | (u64(1) << lane_id());
    return before + (int)__popcll(m & le) - 1;
}

// --- cooperative kernels: workgroup size and the grid barrier ------------

constexpr int kPBlock = 1024;  // 16 waves per CU (up to 128 VGPRs: four waves per SIMD)

struct GridBar {
    Counter group[8];  // arrivals per group (monotonic)
    Counter top;       // completed groups (monotonic)
    Counter rel[8];    // per-group release: the number of the last open barrier
    int32_t fail;
};

// Waits until this wave's memory operations have completed: its device-scope
// stores and atomics have reached the point of coherence.
__device__ __forceinline__ void drain_memory() {
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Two-level barrier, thread 0 of each block; `k` counts the barriers this
// block has passed.  Blocks arrive at one of eight group counters (group g
// holds the blocks of XCD g), the last of each group at the top counter; the
// last of those writes the barrier's number to every group's release word,
// and each block polls its own group's word, so no address takes the polls
// of the whole grid.  Counters only grow, so nothing is reset between
// barriers.  Shared state is only touched through device-scope accesses, so
// draining every wave's outstanding operations before arrival (done by the
// caller for all waves) orders them before the barrier, with no cache
// write-back or invalidation.  A waiter gives up after a bounded spin (the
// kernel then stops with `fail` set) so no bug can hang the device.
__device__ bool grid_arrive_wait(GridBar *B, u64 &k) {
    const unsigned nb = gridDim.x;
    const unsigned g = blockIdx.x & 7;
    const unsigned ngroups = nb < 8 ? nb : 8;
    const unsigned gsize = (nb - g + 7) / 8;
    k += 1;
    if (atomicAdd(&B->group[g].v, 1ull) == k * gsize - 1) {
        if (atomicAdd(&B->top.v, 1ull) == k * ngroups - 1) {
            for (unsigned j = 0; j < ngroups; ++j) st(&B->rel[j].v, k);
        }
    }
    bool ok = true;
    int64_t spins = 0;
    while (ld(&B->rel[g].v) < k) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > (int64_t(1) << 28) || ld(&B->fail)) {
            st(&B->fail, 1);
            ok = false;
            break;
        }
    }
    drain_memory();
    return ok;
}

}  // namespace

}  // namespace bt
