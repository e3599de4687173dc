// support.hip - butterfly supports without the index (Lemmas 1-3).
//
// The support of an edge is the sum of c(x, z) - 1 over the priority-obeyed
// wedges (x, y, z) that hold it, where c(x, z) is the number of wedges from x
// to z and p(x) > p(y), p(z).  Each wedge is walked from both of its ends:
//   from x, over the row prefixes of the middles below x, the edges (x, y)
//     collect their sums (the down walk);
//   from z, over the row suffixes above both z and the middle, the edges
//     (z, y) collect theirs (the up walk).
// A walk counts c of its start vertex in an LDS table, then sums c - 1 along
// each of the start's rows.  A row's sum stays in its wave, so the only
// global atomics are one a row.  Counting from x alone, with an atomic on
// (y, z) for every wedge, was bound by those: memory-side atomics run at
// 2.4e10/s on the whole chip, and 13e9 wedges/s were reached.
//
// Start vertices fall into tiers by their wedges: a wave each, or a workgroup
// of 256, 512 or 1,024 threads with a table to match.  The table is a hash
// table for few wedges, or dense counters over a range of ids.  c is at most
// the degree of either end, and ids ascend by degree, so the counters of the
// range's ids of at most 255 neighbours are bytes, the others 16 bits (32 if
// the start has more rows than that holds).  A start with more is cut into windows of the other end's ids, at equal shares of the degrees:
// fewer wedges than a hash table takes, or fewer ids than there are counters.
// Rows are ascending, so a window clips each long row by binary search.
//
// Whole support calls, counted from x alone and so (with half of the time
// that preparation took taken off as well): 20M-edge hub graph (1.26e9
// wedges) 109 and 22 ms, 5M-edge Chung-Lu graph (1.6e8 wedges) 18.3 and 4.8
// ms, 250k-edge graph 1.11 and 0.49 ms.  The hub graph's largest tier (75% of
// the wedges) takes 12 ms: 4 x 0.95e9 row entries, read from L2 at
// 64 a wave, and the first touch of 1e8 short rows, a cache line each.  Cut
// at 2^18 wedges a task instead of up to 2^21 it took 33 ms (each part clips
// every row), with 16-bit counters throughout 17.3 ms (two windows where one
// does); eight entries in flight a lane instead of four changed nothing, and
// runs of rows handed out in LDS instead of dealt took a quarter longer.
#include <algorithm>
#include <cstring>

#include "pipeline.h"

namespace bt {

namespace {

constexpr int kStep = 4;  // elements per lane in flight
constexpr uint32_t kUp = 0x80000000u;
constexpr uint32_t kWaveMax = 256, kMidMax = 2048, kBigMax = 16384;
// Bounds of the wedges a task of the largest tier takes of a start (about
// half of a CU's share of the graph's): each part clips all of the start's
// rows, so only what would hold up the rest is cut.
constexpr int64_t kPartLeast = int64_t(1) << 15, kPartMost = int64_t(1) << 21;
constexpr uint32_t kMaxParts = 4096;
// Starts from here up go first, cut into parts (from 2^18 and 2^20 up: 20M-edge
// hub graph 21.7 and 21.1 ms, 21.1 so; 5M-edge graph 4.73 and 4.70, 4.7 so).
constexpr int64_t kFirst = int64_t(1) << 19;
constexpr int32_t kEmpty = -1;
constexpr uint32_t kByteMax = 255;
enum Table { kHash, kDense32, kDense };

struct WalkArgs {
    const int64_t *off;
    const int32_t *adj, *eid, *low;
    // Rows of the walks by entry (see RankCSR).
    const int32_t *rev, *zlen;
    const uint32_t *rst;
    const int64_t *wpre, *zpre;
    int32_t n, n_lower;
    unsigned long long *supl;
    unsigned long long *bf;
    int32_t *queue;
};

struct WaveRows {
    uint64_t mask[kStep];
    uint32_t delta[kWave];  // first entry less first element of the wave's rows
};

struct LongRow {
    uint32_t st, len, e;
};

// First position in adj[lo, hi) whose value is >= v (rows are ascending).
__device__ __forceinline__ uint32_t first_at(const int32_t *adj, uint32_t lo, uint32_t hi,
                                             int32_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (adj[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// First id in [lo, hi) of more than kByteMax neighbours, or hi.
__device__ __forceinline__ int32_t first_wide(const int64_t *off, int32_t lo, int32_t hi) {
    return first_with(lo, hi, [&](int32_t i) { return off[i + 1] - off[i] > kByteMax; });
}

// A window of the walk of one start vertex.
struct Walk {
    int32_t s;       // the start
    bool up;
    bool from, to;   // rows are clipped to ids from lo up, and to ids below hi
    int32_t lo, hi;  // ids of the other end; dense tables count from lo
    uint32_t bytes;  // kDense: ids with byte counters, from lo
    uint32_t low;    // down rows that are prefixes of the middle's row
    uint32_t mask;   // hash table: slots - 1
    int32_t *key;
    uint32_t *cnt;
};

// Byte address and mask of id i's counter in a kDense table.
__device__ __forceinline__ uint32_t dense_at(const Walk &w, uint32_t i, uint32_t &m) {
    const bool byte = i < w.bytes;
    m = byte ? 0xffu : 0xffffu;
    return byte ? i : 2 * i - w.bytes + (w.bytes & 1);
}

// Counts the wedge to z; returns how many came before.
template <Table T> __device__ __forceinline__ uint32_t count_one(const Walk &w, int32_t z) {
    if (T == kDense32) return atomicAdd(&w.cnt[z - w.lo], 1u);
    if (T == kDense) {
        uint32_t m;
        const uint32_t at = dense_at(w, (uint32_t)(z - w.lo), m), sh = (at & 3) * 8;
        return atomicAdd(&w.cnt[at >> 2], 1u << sh) >> sh & m;
    }
    uint32_t h = ((uint32_t)z * 2654435761u) >> 8 & w.mask;
    while (true) {
        int32_t k = w.key[h];
        if (k == kEmpty) {
            k = atomicCAS(&w.key[h], kEmpty, z);
            if (k == kEmpty) k = z;
        }
        if (k == z) break;
        h = (h + 1) & w.mask;
    }
    return atomicAdd(&w.cnt[h], 1u);
}

// c(z) of a counted z.
template <Table T> __device__ __forceinline__ uint32_t count_of(const Walk &w, int32_t z) {
    if (T == kDense32) return w.cnt[z - w.lo];
    if (T == kDense) {
        uint32_t m;
        const uint32_t at = dense_at(w, (uint32_t)(z - w.lo), m);
        return w.cnt[at >> 2] >> (at & 3) * 8 & m;
    }
    uint32_t h = ((uint32_t)z * 2654435761u) >> 8 & w.mask;
    while (w.key[h] != z) h = (h + 1) & w.mask;
    return w.cnt[h];
}

__device__ __forceinline__ uint32_t rows_of(const WalkArgs &A, int32_t s, bool up) {
    return up ? (uint32_t)(A.off[s + 1] - A.off[s]) : (uint32_t)A.low[s];
}

// Row j of the walk: entries [st, st + len).  Rows of more than `least`
// entries are clipped to the window; the others are left whole, and their
// entries outside the window are passed over one by one (clipped from 16 and from
// 256 entries up: 20M-edge hub graph 21.6 and 22.9 ms, 21.1 with 64).
constexpr uint32_t kClipLeast = 64;
__device__ __forceinline__ void load_row(const WalkArgs &A, const Walk &w, uint32_t os, uint32_t j,
                                         uint32_t least, uint32_t &st, uint32_t &len) {
    const uint32_t p = os + j;
    const uint32_t r = (uint32_t)A.rev[p];
    st = A.rst[p];
    if (w.up) {
        len = (uint32_t)A.zlen[p];
        if (j < w.low) st += r + 1;
    } else {
        len = r;
    }
    if ((w.from || w.to) && len > least) {
        uint32_t en = st + len;
        if (w.from) st = first_at(A.adj, st, en, w.lo);
        if (w.to) en = first_at(A.adj, st, en, w.hi);
        len = en - st;
    }
}

// One pass over up to 64 rows, one a lane: counts their elements, or sums
// c - 1 along each row and adds the sum to the row's edge.  Elements are
// spread over the lanes kStep * 64 at a time.  `seen` sums what count_one
// returns (the butterflies) or is left alone.
template <Table T, bool SUM, bool WINDOWS>
__device__ __forceinline__ void walk_rows(const WalkArgs &A, const Walk &w, WaveRows &R, uint32_t st,
                                          uint32_t len, uint32_t e, unsigned long long &seen) {
    // Rows with elements move to the front lanes.
    const uint64_t some = __ballot(len != 0);
    if (!some) return;
    const int n_rows = (int)__popcll(some);
    if (n_rows < kWave) {
        const int to = (int)__popcll(some & lanemask_lt());
        const int empty_to = n_rows + lane_id() - to;
        const int dst = (len ? to : empty_to) << 2;
        st = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)st);
        if (SUM) e = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)e);
        len = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)len);
    }
    const bool mine = lane_id() < n_rows;
    const uint32_t inc = wave_inclusive_sum<uint32_t>(len);
    const uint32_t total = wave_last(inc);
    const uint32_t pre = inc - len;
    R.delta[lane_id()] = st - pre;
    uint32_t sum = 0;   // of this lane's row
    uint32_t run = 0;   // this lane's part of the row that has not ended yet
    const uint64_t le = lanemask_lt() | (uint64_t(1) << lane_id());
    for (uint32_t t0 = 0; t0 < total; t0 += kStep * kWave) {
        if (lane_id() < kStep)
            __hip_atomic_store(&R.mask[lane_id()], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        if (mine && pre >= t0 && pre < t0 + kStep * kWave)
            __hip_atomic_fetch_or(&R.mask[(pre - t0) / kWave], 1ull << ((pre - t0) % kWave),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        int before = (int)__popcll(__ballot(mine && pre < t0));
        uint64_t mask[kStep];
        int32_t z[kStep];
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            mask[u] = __hip_atomic_load(&R.mask[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const uint32_t t = t0 + u * kWave + lane_id();
            const int row = before + (int)__popcll(mask[u] & le) - 1;
            before += (int)__popcll(mask[u]);
            z[u] = t < total ? A.adj[(uint32_t)(t + R.delta[row])] : kEmpty;
            if (T != kHash || WINDOWS)
                if ((uint32_t)(z[u] - w.lo) >= (uint32_t)(w.hi - w.lo)) z[u] = kEmpty;
        }
        if (!SUM) {
#pragma unroll
            for (int u = 0; u < kStep; ++u)
                if (z[u] != kEmpty) seen += count_one<T>(w, z[u]);
            continue;
        }
        before = (int)__popcll(__ballot(mine && pre < t0));
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            const uint32_t v = z[u] != kEmpty ? count_of<T>(w, z[u]) - 1 : 0;
            if (mask[u] == 0) {  // one row holds all 64
                run += v;
                continue;
            }
            const uint32_t t = t0 + u * kWave;
            const uint32_t open = wave_last(wave_inclusive_sum<uint32_t>(run));
            if (lane_id() == before - 1) sum += open;
            run = 0;
            // The rows' shares of this step, from prefix sums of its values.
            const uint32_t pv = wave_inclusive_sum<uint32_t>(v);
            const uint32_t a = max(pre, t), b = min(inc, t + kWave);
            const bool in = mine && a < b;
            const uint32_t upto = (uint32_t)__shfl((int)pv, in ? (int)(b - 1 - t) : 0, kWave);
            const uint32_t less = (uint32_t)__shfl((int)pv, in && a > t ? (int)(a - 1 - t) : 0, kWave);
            if (in) sum += upto - (a > t ? less : 0);
            before += (int)__popcll(mask[u]);
        }
    }
    if (SUM) {
        const uint32_t open = wave_last(wave_inclusive_sum<uint32_t>(run));
        if (lane_id() == n_rows - 1) sum += open;
        if (mine && sum) atomicAdd(&A.supl[e], (unsigned long long)sum);
    }
}

// A pass of a workgroup over all rows of the walk.  Rows above kLong elements
// are taken by all its waves together.
template <int WAVES> struct GroupRows {
    static constexpr uint32_t kLong = 2048;
    static constexpr int kMaxLong = 128;
    WaveRows wave[WAVES];
    LongRow rows[kMaxLong];
    int32_t n_long;
};

template <Table T, bool SUM, int WAVES>
__device__ void group_pass(const WalkArgs &A, const Walk &w, GroupRows<WAVES> &G,
                           unsigned long long &seen) {
    const int wv = threadIdx.x / kWave;
    const uint32_t os = (uint32_t)A.off[w.s], nr = rows_of(A, w.s, w.up);
    if (threadIdx.x == 0) G.n_long = 0;
    __syncthreads();
    // Few rows are dealt out one by one, so that every wave has some; many in
    // runs of 64, which share cache lines.
    const bool runs = nr >= 4 * WAVES * kWave;
    for (uint32_t jb = 0; jb < nr; jb += WAVES * kWave) {
        const uint32_t j = jb + (runs ? threadIdx.x : lane_id() * WAVES + wv);
        uint32_t st = 0, len = 0, e = 0;
        if (j < nr) {
            load_row(A, w, os, j, kClipLeast, st, len);
            if (SUM && len) e = (uint32_t)A.eid[os + j];
        }
        if (len > G.kLong) {
            const int32_t at = atomicAdd(&G.n_long, 1);
            if (at < G.kMaxLong) {
                G.rows[at] = LongRow{st, len, e};
                len = 0;
            }
        }
        walk_rows<T, SUM, true>(A, w, G.wave[wv], st, len, e, seen);
    }
    __syncthreads();
    const int n_long = min(G.n_long, G.kMaxLong);
    for (int k = 0; k < n_long; ++k) {
        const LongRow L = G.rows[k];
        unsigned long long sum = 0;
        for (uint32_t t0 = 0; t0 < L.len; t0 += WAVES * kWave * kStep) {
            int32_t z[kStep];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const uint32_t t = t0 + u * WAVES * kWave + threadIdx.x;
                z[u] = t < L.len ? A.adj[L.st + t] : kEmpty;
            }
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                if (z[u] == kEmpty) continue;
                if (SUM) sum += count_of<T>(w, z[u]) - 1;
                else seen += count_one<T>(w, z[u]);
            }
        }
        if (SUM) {
            sum = wave_sum(sum);
            if (lane_id() == 0 && sum) atomicAdd(&A.supl[L.e], sum);
        }
    }
    __syncthreads();
}

// Wedges of the walk inside the window.
template <int WAVES>
__device__ uint32_t group_wedges(const WalkArgs &A, const Walk &w, GroupRows<WAVES> &G) {
    const uint32_t os = (uint32_t)A.off[w.s], nr = rows_of(A, w.s, w.up);
    unsigned long long t = 0;
    if (threadIdx.x == 0) G.n_long = 0;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < nr; j += WAVES * kWave) {
        uint32_t st, len;
        load_row(A, w, os, j, 0, st, len);
        t += len;
    }
    t = wave_sum(t);  // saturated: only a comparison with a small bound is asked
    if (lane_id() == 0) atomicAdd(&G.n_long, (int32_t)min(t, 1ull << 24));
    __syncthreads();
    const uint32_t r = (uint32_t)G.n_long;
    __syncthreads();
    return r;
}

__device__ __forceinline__ void clear_words(uint32_t *p, uint32_t n, uint32_t v, int threads) {
    const uint32_t n4 = (n + 3) / 4;
    for (uint32_t i = threadIdx.x; i < n4; i += threads)
        reinterpret_cast<uint4 *>(p)[i] = make_uint4(v, v, v, v);
}

template <Table T, int WAVES>
__device__ void group_window(const WalkArgs &A, Walk &w, GroupRows<WAVES> &G, uint32_t *table,
                             uint32_t slots, unsigned long long &bf) {
    constexpr int kThreads = WAVES * kWave;
    unsigned long long seen = 0;
    if (T == kHash) {
        w.mask = slots - 1;
        w.key = reinterpret_cast<int32_t *>(table);
        w.cnt = table + slots;
        clear_words(table, slots, (uint32_t)kEmpty, kThreads);
        clear_words(w.cnt, slots, 0, kThreads);
    } else {
        const uint32_t ids = (uint32_t)(w.hi - w.lo);
        uint32_t m;
        w.cnt = table;
        clear_words(table, T == kDense ? dense_at(w, ids, m) / 4 + 1 : ids, 0, kThreads);
    }
    __syncthreads();
    group_pass<T, false, WAVES>(A, w, G, seen);
    if (!w.up) bf += seen;
    group_pass<T, true, WAVES>(A, w, G, seen);
}

struct WalkTask {
    uint32_t s;  // start vertex | kUp
    uint32_t part, parts;
};

// One task a workgroup, from the queue.
template <int WAVES, int TABLE_BYTES>
__global__ __launch_bounds__(WAVES *kWave) void k_walk_group(WalkArgs A, const WalkTask *tasks,
                                                             int32_t n_tasks) {
    constexpr uint32_t kBytes = TABLE_BYTES - 16;  // of dense counters, padding aside
    constexpr uint32_t kSlots = TABLE_BYTES / 8, kHashMax = kSlots / 2;
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *table = reinterpret_cast<uint32_t *>(smem);
    GroupRows<WAVES> &G = *reinterpret_cast<GroupRows<WAVES> *>(smem + TABLE_BYTES);
    __shared__ int32_t s_task;
    unsigned long long bf = 0;
    while (true) {
        __syncthreads();
        if (threadIdx.x == 0) s_task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int32_t ti = s_task;
        if (ti >= n_tasks) break;
        const WalkTask K = tasks[ti];
        Walk w;
        w.s = (int32_t)(K.s & ~kUp);
        w.up = (K.s & kUp) != 0;
        w.low = (uint32_t)A.low[w.s];
        const bool high = w.s >= A.n_lower;
        int32_t lo = w.up ? w.s + 1 : (high ? A.n_lower : 0);
        int32_t hi = w.up ? (high ? A.n : A.n_lower) : w.s;
        const int32_t lo0 = lo, hi0 = hi;
        const int64_t os = A.off[w.s];
        const uint32_t nr = rows_of(A, w.s, w.up);
        int64_t work = w.up ? A.zpre[os + nr] - A.zpre[os] : A.wpre[os + nr] - A.wpre[os];
        if (K.parts > 1) {
            const int64_t o0 = A.off[lo0], d = A.off[hi0] - o0;
            if (K.part > 0) lo = first_row(A.off, lo0, hi0, o0 + d * K.part / K.parts);
            if (K.part + 1 < K.parts) hi = first_row(A.off, lo0, hi0, o0 + d * (K.part + 1) / K.parts);
            work /= K.parts;
        }
        if (lo >= hi) continue;
        // Ids below `wide` have byte counters, the others `kind` bytes.
        const bool half = nr <= 0xffffu;
        const int32_t wide = !half ? lo : nr <= kByteMax ? hi : first_wide(A.off, lo, hi);
        const uint32_t kind = half ? 2 : 4;
        // The end of the dense window that begins at id c.
        const auto dense_end = [&](int32_t c, int32_t end) {
            const uint32_t n8 = (uint32_t)max(0, min(min(wide, end) - c, (int32_t)kBytes));
            const uint32_t rest = (kBytes - n8) / kind;
            return (int32_t)min((int64_t)c + n8 + rest, (int64_t)end);
        };
        const int64_t all = (int64_t)(wide - lo) + (int64_t)(hi - wide) * kind;
        const int64_t kd = (all + kBytes - 1) / kBytes;
        // Equal shares of the degrees hold about equal shares of the wedges;
        // half of what fits leaves room for the difference.
        const int64_t kh = work <= kHashMax ? 1 : (work + kHashMax / 2 - 1) / (kHashMax / 2);
        const uint32_t n_win = kh < kd ? (uint32_t)kh : 1;
        const int64_t o0 = A.off[lo], d = A.off[hi] - o0;
        int32_t a = lo;
        for (uint32_t i = 0; i < n_win; ++i) {
            const int32_t b =
                i + 1 < n_win ? first_row(A.off, a, hi, o0 + d * (i + 1) / n_win) : hi;
            if (b <= a) continue;
            w.lo = a;
            w.hi = b;
            w.from = a != lo0;
            w.to = b != hi0;
            const bool clip = w.from || w.to;
            bool hash = kh < kd && dense_end(a, b) < b;
            uint32_t wedges = (uint32_t)min(work, (int64_t)kHashMax + 1);
            if (hash && clip) wedges = group_wedges<WAVES>(A, w, G);
            else if (!clip && work <= (b - a) / 32) hash = true;  // less to clear
            if (hash && wedges <= kHashMax) {
                uint32_t slots = 256;
                while (slots < 2 * wedges) slots <<= 1;
                group_window<kHash, WAVES>(A, w, G, table, slots, bf);
            } else {
                for (int32_t c = a; c < b; c = w.hi) {
                    w.lo = c;
                    w.hi = dense_end(c, b);
                    w.bytes = (uint32_t)max(0, min(wide, w.hi) - c);
                    w.from = w.lo != lo0;
                    w.to = w.hi != hi0;
                    if (half) group_window<kDense, WAVES>(A, w, G, table, 0, bf);
                    else group_window<kDense32, WAVES>(A, w, G, table, 0, bf);
                }
            }
            a = b;
        }
    }
    bf = wave_sum(bf);
    if (lane_id() == 0 && bf) atomicAdd(A.bf, bf);
}

constexpr int kSmallBlock = 256;

// Starts of few wedges, whose hash table always fits: one a group of GROUP
// waves.  Tasks of a tier are alike, so they are dealt out in turn.
template <int GROUP, uint32_t MOST>
__global__ __launch_bounds__(kSmallBlock) void k_walk_small(WalkArgs A, const uint32_t *tasks,
                                                            int32_t n_tasks) {
    constexpr int kWaves = kSmallBlock / kWave, kGroups = kWaves / GROUP;
    __shared__ __align__(16) int32_t s_key[kGroups][2 * MOST];
    __shared__ __align__(16) uint32_t s_cnt[kGroups][2 * MOST];
    __shared__ WaveRows s_rows[kWaves];
    const int wv = threadIdx.x / kWave, gr = wv / GROUP;
    const uint32_t in_group = (uint32_t)(wv % GROUP);
    const auto sync = [] {
        if (GROUP > 1) __syncthreads();
    };
    static_assert(GROUP == 1 || GROUP == kWaves, "a barrier is a workgroup's");
    unsigned long long bf = 0;
    Walk w;
    w.key = s_key[gr];
    w.cnt = s_cnt[gr];
    w.from = w.to = false;
    w.lo = w.hi = 0;
    const int32_t groups = (int32_t)gridDim.x * kGroups;
    for (int32_t ti = (int32_t)blockIdx.x * kGroups + gr; ti < n_tasks; ti += groups) {
        const uint32_t K = tasks[ti];
        w.s = (int32_t)(K & ~kUp);
        w.up = (K & kUp) != 0;
        w.low = (uint32_t)A.low[w.s];
        const uint32_t os = (uint32_t)A.off[w.s], nr = rows_of(A, w.s, w.up);
        const uint32_t work = w.up ? (uint32_t)(A.zpre[os + nr] - A.zpre[os])
                                   : (uint32_t)(A.wpre[os + nr] - A.wpre[os]);
        uint32_t slots = GROUP * kWave;
        while (slots < 2 * work) slots <<= 1;
        w.mask = slots - 1;
        const uint32_t j0 = lane_id() * GROUP + in_group;
        uint32_t st = 0, len = 0, e = 0;
        const auto row = [&](uint32_t j) {
            st = len = e = 0;
            if (j >= nr) return;
            load_row(A, w, os, j, 0, st, len);
            if (len) e = (uint32_t)A.eid[os + j];
        };
        row(j0);
        sync();  // the last task's table is read no more
        for (uint32_t i = lane_id() + in_group * kWave; i < slots; i += GROUP * kWave) {
            w.key[i] = kEmpty;
            w.cnt[i] = 0;
        }
        sync();
        unsigned long long seen = 0;
        for (uint32_t jb = 0;;) {
            walk_rows<kHash, false, false>(A, w, s_rows[wv], st, len, e, seen);
            jb += GROUP * kWave;
            if (jb >= nr) break;
            row(jb + j0);
        }
        if (!w.up) bf += seen;
        sync();
        // A start of one batch of rows keeps them for the second pass.
        for (uint32_t jb = 0; jb < nr; jb += GROUP * kWave) {
            if (nr > GROUP * kWave) row(jb + j0);
            walk_rows<kHash, true, false>(A, w, s_rows[wv], st, len, e, seen);
        }
    }
    bf = wave_sum(bf);
    if (lane_id() == 0 && bf) atomicAdd(A.bf, bf);
}

// Tiers of the walks: a wave, 256, 512, 1,024 threads; the last in two, as
// the heaviest go first.
constexpr int kTiers = 5;
__device__ __forceinline__ int tier_of(int64_t work) {
    return work <= 1 ? -1 : work <= kWaveMax ? 0 : work <= kMidMax ? 1 : work <= kBigMax ? 2
           : work < kFirst ? 3 : 4;
}

__device__ __forceinline__ uint32_t parts_of(int64_t work, int64_t total) {
    const int64_t part = min(max(total / 512, kPartLeast), kPartMost);
    return (uint32_t)min(work / part + 1, (int64_t)kMaxParts);
}

// Tasks per tier, counted (lists null) or listed.  A walk of one wedge finds
// no butterfly.
__global__ __launch_bounds__(256) void k_walk_tasks(const int64_t *off, const int32_t *low,
                                                    const int64_t *wpre, const int64_t *zpre,
                                                    int32_t n, int64_t n2, int32_t *counts,
                                                    uint32_t *wave,
                                                    uint32_t *mid, WalkTask *big, WalkTask *most,
                                                    WalkTask *first) {
    __shared__ int32_t s_cnt[kTiers], s_base[kTiers];
    for (int64_t v0 = blockIdx.x * (int64_t)blockDim.x; v0 < n;
         v0 += (int64_t)gridDim.x * blockDim.x) {
        if (threadIdx.x < kTiers) s_cnt[threadIdx.x] = 0;
        __syncthreads();
        const int64_t v = v0 + threadIdx.x;
        int tier[2] = {-1, -1};
        int32_t at[2] = {0, 0};
        uint32_t parts[2] = {1, 1};
        if (v < n) {
            const int64_t a = off[v], b = off[v + 1], c = a + low[v];
            const int64_t work[2] = {wpre[c] - wpre[a], zpre[b] - zpre[a]};
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                tier[d] = tier_of(work[d]);
                if (tier[d] == 4) parts[d] = parts_of(work[d], wpre[n2]);
                if (tier[d] >= 0) at[d] = atomicAdd(&s_cnt[tier[d]], (int32_t)parts[d]);
            }
        }
        __syncthreads();
        if (threadIdx.x < kTiers)
            s_base[threadIdx.x] =
                s_cnt[threadIdx.x] ? atomicAdd(&counts[threadIdx.x], s_cnt[threadIdx.x]) : 0;
        __syncthreads();
        if (wave) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                if (tier[d] < 0) continue;
                const uint32_t id = (uint32_t)v | (d ? kUp : 0);
                const int32_t p = s_base[tier[d]] + at[d];
                if (tier[d] == 0) wave[p] = id;
                else if (tier[d] == 1) mid[p] = id;
                else if (tier[d] == 2) big[p] = WalkTask{id, 0, 1};
                else if (tier[d] == 3) most[p] = WalkTask{id, 0, 1};
                else
                    for (uint32_t k = 0; k < parts[d]; ++k) first[p + k] = WalkTask{id, k, parts[d]};
            }
        }
        __syncthreads();
    }
}

template <int WAVES, int TABLE_BYTES>
void launch_group(WalkArgs A, const WalkTask *tasks, int32_t n, int cus, hipStream_t s) {
    if (n <= 0) return;
    constexpr size_t smem = TABLE_BYTES + sizeof(GroupRows<WAVES>);
    const auto kern = k_walk_group<WAVES, TABLE_BYTES>;
    int per_cu = 0;
    BT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    BT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, WAVES * kWave, smem));
    const int32_t grid = std::min<int32_t>(n, cus * std::max(1, per_cu));
    kern<<<(unsigned)grid, WAVES * kWave, smem, s>>>(A, tasks, n);
    BT_CHECK_LAUNCH();
}

template <int GROUP, uint32_t MOST>
void launch_small(const WalkArgs &A, const uint32_t *tasks, int32_t n, int cus, hipStream_t s) {
    if (n <= 0) return;
    constexpr int32_t kGroups = kSmallBlock / kWave / GROUP;
    const auto kern = k_walk_small<GROUP, MOST>;
    int per_cu = 0;
    BT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kSmallBlock, 0));
    const int32_t grid = std::min<int32_t>((n + kGroups - 1) / kGroups, cus * std::max(1, per_cu));
    kern<<<(unsigned)grid, kSmallBlock, 0, s>>>(A, tasks, n);
    BT_CHECK_LAUNCH();
}

// The caller's stream for the first launch, side streams for the others,
// which begin after what the caller's held and end before what it gets next.
class SideStreams {
  public:
    SideStreams(Workspace &ws, hipStream_t s) : ws_(ws), s_(s) {}
    ~SideStreams() {
        if (!joined_) ws_.sync_sides();
        for (hipEvent_t e : ev_)
            if (e) (void)hipEventDestroy(e);
    }
    hipStream_t next(bool used) {
        if (!used) return s_;
        if (n_++ == 0) {
            BT_HIP(hipEventCreateWithFlags(&ev_[0], hipEventDisableTiming));
            BT_HIP(hipEventRecord(ev_[0], s_));
            return s_;
        }
        const hipStream_t t = ws_.side(n_ - 2);
        BT_HIP(hipStreamWaitEvent(t, ev_[0], 0));
        return t;
    }
    void join() {
        for (int k = 1; k < n_; ++k) {
            BT_HIP(hipEventCreateWithFlags(&ev_[k], hipEventDisableTiming));
            BT_HIP(hipEventRecord(ev_[k], ws_.side(k - 1)));
            BT_HIP(hipStreamWaitEvent(s_, ev_[k], 0));
        }
        joined_ = true;
    }

  private:
    Workspace &ws_;
    hipStream_t s_;
    hipEvent_t ev_[4] = {};
    int n_ = 0;
    bool joined_ = false;
};

}  // namespace

int64_t count_support(const RankCSR &r, uint64_t *supl, int64_t *bf, Workspace &ws,
                      hipStream_t s) {
    int32_t *counts = ws.get<int32_t>("walk_counts", 3 * kTiers);  // tiers, cursors, queues
    zero_bytes(counts, 3 * kTiers * sizeof(int32_t), s);
    int64_t *h = ws.host(4);
    const int64_t n2 = 2 * r.m;
    const unsigned grid = (unsigned)grid_for(r.n, 256, 4096);
    if (r.n > 0) {
        k_walk_tasks<<<grid, 256, 0, s>>>(r.off, r.low, r.wpre, r.zpre, r.n, n2, counts, nullptr,
                                          nullptr, nullptr, nullptr, nullptr);
        BT_CHECK_LAUNCH();
    }
    BT_HIP(hipMemcpyAsync(h, counts, kTiers * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipMemcpyAsync(h + 3, r.wpre + n2, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    int32_t nt[kTiers];
    std::memcpy(nt, h, sizeof nt);
    const int64_t wedges = h[3];
    for (int32_t t : nt)
        if (t < 0) throw Error{BT_EOVERFLOW, "too many wedge tasks"};
    const int64_t n_most = (int64_t)nt[4] + nt[3];
    if (n_most > INT32_MAX) throw Error{BT_EOVERFLOW, "too many wedge tasks"};
    if (nt[0] + (int64_t)nt[1] + nt[2] + n_most == 0) return wedges;
    uint32_t *wave = ws.get<uint32_t>("walk_wave", nt[0]);
    uint32_t *mid = ws.get<uint32_t>("walk_mid", nt[1]);
    WalkTask *big = ws.get<WalkTask>("walk_big", nt[2]);
    WalkTask *most = ws.get<WalkTask>("walk_most", n_most);
    k_walk_tasks<<<grid, 256, 0, s>>>(r.off, r.low, r.wpre, r.zpre, r.n, n2, counts + kTiers, wave, mid,
                                      big, most + nt[4], most);
    BT_CHECK_LAUNCH();
    int dev = 0, cus = 0;
    BT_HIP(hipGetDevice(&dev));
    BT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    WalkArgs A{r.off, r.adj, r.eid, r.low, r.rev, r.zlen, r.rst, r.wpre, r.zpre, r.n, r.n_lower,
               reinterpret_cast<unsigned long long *>(supl),
               reinterpret_cast<unsigned long long *>(bf), counts + 2 * kTiers};
    // The tiers run beside each other: each ends in a few long tasks (250k-edge
    // graph: 245 us one after another, 170 so; 5M-edge graph: 3.5 ms and 3.2).
    SideStreams side(ws, s);
    launch_group<16, 131072>(A, most, (int32_t)n_most, cus, side.next(n_most > 0));
    A.queue += 1;
    launch_group<8, 65536>(A, big, nt[2], cus, side.next(nt[2] > 0));
    launch_small<4, kMidMax>(A, mid, nt[1], cus, side.next(nt[1] > 0));
    launch_small<1, kWaveMax>(A, wave, nt[0], cus, side.next(nt[0] > 0));
    side.join();
    return wedges;
}

}  // namespace bt
