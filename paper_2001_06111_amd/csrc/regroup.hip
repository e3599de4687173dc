// regroup.hip - from a swept depth to the next: the edges, wedges and blooms
// of each part put together.
//
// A part's peel needs the wedges whose first-removed edge lies in the part,
// that is, whose smaller part among its two edges is this one: each wedge
// belongs to exactly one part, so all parts together hold the index once.
// Within a part, the wedges of one bloom form a bloom of their own whose
// bloom number starts at what the bloom had when the part began (its wedges
// of later parts still count, but none of their edges is touched).
//
// Edges are sorted by part (stable: the locality order survives).  Wedges of
// parts of a single level are done; the others are compacted in bloom order
// and sorted by part (stable), so each part's wedges are contiguous and, in
// them, each bloom's.
#include <climits>

#include "peel_split.h"

namespace bt {

namespace {

constexpr uint32_t kLeafWedges = 500000;
constexpr int kLeafMostLog2 = 22;  // of the wedges of any leaf
static_assert((int64_t(1) << kLeafMostLog2) <= kLeafJobWedges, "a leaf's work items hold them");
constexpr int kTile = 2048;  // wedges per tile of the order-keeping compactions

__global__ void k_edge_keys(const EdgeMark *mark, int64_t m, int32_t n_parts, uint64_t *keys,
                            uint32_t *vals) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = mark_part(mark[e].v);
        keys[e] = (uint64_t)(p < 0 || p >= n_parts ? n_parts : p);
        vals[e] = (uint32_t)e;
    }
}

// [first[p], last[p]) of each part in the sorted edges (cleared before).
__global__ void k_part_bounds(const uint64_t *keys, int64_t m, int64_t *first, int64_t *last) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[i];
        if (i == 0 || keys[i - 1] != k) first[k] = i;
        if (i == m - 1 || keys[i + 1] != k) last[k] = i + 1;
    }
}

// Where a part's edges go: base >= 0, the new id of its first (of a job, or,
// from rank n_jobs on, of a leaf in the pool); base < 0: its edges are done,
// at level ~base.  rank: its place in the wedges' order.
struct PartMap {
    int32_t base;
    uint32_t rank;
};

__global__ void k_renumber(const uint64_t *keys, const uint32_t *vals, int64_t n,
                           const PartMap *map, const int64_t *first, const int32_t *oid,
                           int32_t *newid, uint32_t n_jobs, int32_t *oid_jobs,
                           int32_t *oid_pool, int64_t *phi_out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t p = keys[i];
        const uint32_t e = vals[i];
        const int32_t o = oid ? oid[e] : (int32_t)e;
        const PartMap M = map[p];
        if (M.base < 0) {
            phi_out[o] = ~M.base;
        } else {
            const int32_t id = M.base + (int32_t)(i - first[p]);
            newid[e] = id;
            (M.rank < n_jobs ? oid_jobs : oid_pool)[id] = o;
        }
    }
}

// The part each wedge belongs to, the smaller one of its two edges' (n_parts:
// none, an edge of no part here is never removed), and the parts' wedges.
// Counted in LDS where the counts fit.
template <bool LDS>
__global__ __launch_bounds__(1024) void k_wedge_parts(const int32_t *wea, const int32_t *web,
                                                      int64_t nw, const EdgeMark *mark,
                                                      int32_t n_parts, int32_t *wpart,
                                                      uint32_t *count) {
    extern __shared__ uint32_t s_cnt[];
    if (LDS) {
        for (int i = threadIdx.x; i <= n_parts; i += blockDim.x) s_cnt[i] = 0;
        __syncthreads();
    }
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < nw;
         w += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t a = (uint32_t)wea[w], b = (uint32_t)web[w];
        const int32_t pa = a & kFixedBit ? INT_MAX : mark_part(mark[a].v);
        const int32_t pb = b & kFixedBit ? INT_MAX : mark_part(mark[b].v);
        const int32_t p = min(min(pa, pb), n_parts);
        wpart[w] = p;
        atomicAdd(LDS ? &s_cnt[p] : &count[p], 1u);
    }
    if (LDS) {
        __syncthreads();
        for (int i = threadIdx.x; i <= n_parts; i += blockDim.x)
            if (s_cnt[i]) atomicAdd(&count[i], s_cnt[i]);
    }
}
constexpr int32_t kLdsParts = 12288;

__global__ __launch_bounds__(256) void k_keep_count(const int32_t *wpart, int64_t nw,
                                                    const PartMap *map, uint32_t n_ranks,
                                                    int32_t *tile) {
    __shared__ int32_t s_c;
    for (int64_t t = blockIdx.x; t * kTile < nw; t += gridDim.x) {
        if (threadIdx.x == 0) s_c = 0;
        __syncthreads();
        int32_t c = 0;
        for (int k = threadIdx.x; k < kTile; k += 256) {
            const int64_t w = t * kTile + k;
            if (w < nw && map[wpart[w]].rank < n_ranks) ++c;
        }
        c = wave_sum(c);
        if (lane_id() == 0 && c) atomicAdd(&s_c, c);
        __syncthreads();
        if (threadIdx.x == 0) tile[t] = s_c;
        __syncthreads();
    }
}

// Kept wedges in bloom order: key (bloom, rank), value the wedge.
__global__ __launch_bounds__(256) void k_keep_write(const int32_t *wpart, const int32_t *wbl,
                                                    int64_t nw, const PartMap *map,
                                                    uint32_t n_ranks, const int64_t *tile_off,
                                                    uint64_t *keys, uint32_t *vals) {
    __shared__ uint32_t s_w[256 / kWave + 1];
    for (int64_t t = blockIdx.x; t * kTile < nw; t += gridDim.x) {
        int64_t base = tile_off[t];
        for (int k0 = 0; k0 < kTile; k0 += 256) {
            const int64_t w = t * kTile + k0 + threadIdx.x;
            const uint32_t r = w < nw ? map[wpart[w]].rank : 0xffffffffu;
            const bool keep = r < n_ranks;
            uint32_t total;
            const uint32_t pre = block_exclusive_sum<uint32_t>(keep ? 1u : 0u, s_w, &total);
            if (keep) {
                keys[base + pre] = ((uint64_t)(uint32_t)wbl[w] << 32) | r;
                vals[base + pre] = (uint32_t)w;
            }
            base += total;
        }
    }
}

__device__ __forceinline__ bool is_head(const uint64_t *keys, int64_t i) {
    return i == 0 || keys[i] != keys[i - 1];
}

__global__ __launch_bounds__(256) void k_head_count(const uint64_t *keys, int64_t n,
                                                    int32_t *tile) {
    __shared__ int32_t s_c;
    for (int64_t t = blockIdx.x; t * kTile < n; t += gridDim.x) {
        if (threadIdx.x == 0) s_c = 0;
        __syncthreads();
        int32_t c = 0;
        for (int k = threadIdx.x; k < kTile; k += 256) {
            const int64_t i = t * kTile + k;
            if (i < n && is_head(keys, i)) ++c;
        }
        c = wave_sum(c);
        if (lane_id() == 0 && c) atomicAdd(&s_c, c);
        __syncthreads();
        if (threadIdx.x == 0) tile[t] = s_c;
        __syncthreads();
    }
}

// An edge as the wedge's part sees it.
__device__ __forceinline__ int32_t edge_in(uint32_t e, uint32_t rank, const EdgeMark *mark,
                                           const PartMap *map, const int32_t *newid) {
    if (e & kFixedBit) return (int32_t)kFixedBit;
    const int32_t p = mark_part(mark[e].v);
    if (p == INT_MAX || map[p].rank != rank) return (int32_t)kFixedBit;
    return newid[e];
}

// Wedge and bloom arrays of the jobs or of the pool.
struct Dest {
    int32_t *wea, *web, *wbl, *bk;
    uint32_t *bwoff;
    int64_t w, b;  // position of the first sorted wedge and bloom
};

// The sorted wedges' records, their blooms, and the blooms' numbers: what one
// killed wedge of the bloom carries (blooms of wedges that outlived theirs in
// the sweep carry none and hold no butterfly).  The first nw_jobs wedges are
// the jobs', the others leaves'.
__global__ __launch_bounds__(256) void k_build(const uint64_t *keys, const uint32_t *vals,
                                               int64_t n, int64_t nw_jobs, const int64_t *tile_off,
                                               const int32_t *wea, const int32_t *web,
                                               const int32_t *wedge_k, const EdgeMark *mark,
                                               const PartMap *map, const int32_t *newid, Dest J,
                                               Dest L) {
    __shared__ uint32_t s_w[256 / kWave + 1];
    for (int64_t t = blockIdx.x; t * kTile < n; t += gridDim.x) {
        int64_t base = tile_off[t];
        for (int k0 = 0; k0 < kTile; k0 += 256) {
            const int64_t i = t * kTile + k0 + threadIdx.x;
            const bool head = i < n && is_head(keys, i);
            uint32_t total;
            const uint32_t pre = block_exclusive_sum<uint32_t>(head ? 1u : 0u, s_w, &total);
            if (i < n) {
                const Dest &D = i < nw_jobs ? J : L;
                const int64_t b = D.b + base + pre + (head ? 1 : 0) - 1, x = D.w + i;
                const uint32_t w = vals[i], rank = (uint32_t)keys[i];
                D.wea[x] = edge_in((uint32_t)wea[w], rank, mark, map, newid);
                D.web[x] = edge_in((uint32_t)web[w], rank, mark, map, newid);
                D.wbl[x] = (int32_t)b;
                if (head) D.bwoff[b] = (uint32_t)x;
                const int32_t kw = wedge_k[w];
                if (kw > 0) D.bk[b] = kw;
            }
            base += total;
        }
        __syncthreads();
    }
}

__device__ __forceinline__ int64_t rank_start(const uint64_t *keys, int64_t n, uint32_t rank) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((uint32_t)keys[mid] < rank) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// First wedge and bloom of the ranks from n_jobs to n_ranks (one entry more
// than the leaves): where the heads are counted by tile, a rank's first bloom
// is the heads before its first wedge.  One wave a rank.
__global__ __launch_bounds__(256) void k_rank_bounds(const uint64_t *keys, int64_t n,
                                                     const int64_t *tile_off, int32_t n_jobs,
                                                     int32_t n_ranks, int64_t *bounds) {
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t j = n_jobs + (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
         j <= n_ranks; j += nw) {
        const int64_t w = rank_start(keys, n, (uint32_t)j);
        int64_t heads = 0;
        for (int64_t i = (w / kTile) * kTile + lane_id(); i < w; i += kWave)
            heads += is_head(keys, i) ? 1 : 0;
        heads = wave_sum(heads);
        if (lane_id() == 0) {
            bounds[2 * (j - n_jobs)] = w;
            bounds[2 * (j - n_jobs) + 1] = tile_off[w / kTile] + heads;
        }
    }
}

__global__ void k_put_u32(uint32_t *p, uint32_t v) { *p = v; }

// Supports and link counts of the jobs' edges, as the index build packs them.
__global__ void k_job_supports(const int32_t *wea, const int32_t *web, const int32_t *wbl,
                               const int32_t *bk, int64_t nw, unsigned long long *supl) {
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < nw;
         w += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t a = (uint32_t)wea[w], b = (uint32_t)web[w];
        const int32_t k = bk[wbl[w]];
        const unsigned long long add = (1ull << 32) | (uint32_t)max(k - 1, 0);
        if (!(a & kFixedBit)) atomicAdd(&supl[a], add);
        if (!(b & kFixedBit)) atomicAdd(&supl[b], add);
    }
}

__global__ void k_job_link_counts(const uint64_t *supl, int64_t m, int32_t *cnt) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x)
        cnt[e] = (int32_t)(supl[e] >> 32);
}

__global__ void k_job_links(const int32_t *wea, const int32_t *web, const int32_t *wbl, int64_t nw,
                            unsigned long long *supl, const int64_t *link_off, uint3 *link) {
    const unsigned long long one = 1ull << 32;
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < nw;
         w += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t a = (uint32_t)wea[w], b = (uint32_t)web[w], bl = (uint32_t)wbl[w];
        if (!(a & kFixedBit)) {
            const unsigned long long o = atomicAdd(&supl[a], 0ull - one);
            link[link_off[a] + (int64_t)(o >> 32) - 1] = make_uint3((uint32_t)w, bl, b);
        }
        if (!(b & kFixedBit)) {
            const unsigned long long o = atomicAdd(&supl[b], 0ull - one);
            link[link_off[b] + (int64_t)(o >> 32) - 1] = make_uint3((uint32_t)w, bl, a);
        }
    }
}

// Whether a part is peeled by one workgroup.  A leaf takes about 60 ns a
// wedge, which a sweep that splits it further must beat: with 250,000 and
// 1,000,000 wedges in place of kLeafWedges 249 and 223 ms (5M-edge graph, 229 as
// it is), 150 and 131 (192 pool graphs, 135), 102 and 103 (400,000-edge hub graph
// by BiT-PC, 98), 225 and 220 (2M-edge hub graph, 214).  Parts that a sweep took
// whole, or that several have not brought down, are left to it as well; so are
// parts of a few hundred edges, which a sweep's rounds and launches would cost
// more (each of these two changes none of the above by 1%, at 0 to 8,192 edges
// and depths 2 to 100).
// Above `most` wedges a part goes on to the next sweep whatever it is: its
// positions must fit the work items, and one workgroup would take seconds.  A
// part that a sweep took whole is cut by levels, whose range shrinks by 16 a
// depth, down to single ones, so it ends.  Bounds of 2^20, 2^22 and 2^25: 2M-edge
// request graph 514, 527 and 543 ms (its largest leaves 0.7, 2.6 and 4.2 million
// wedges), 20M-edge hub graph 2.94, 2.91 and 2.92 s (1.0, 1.6 and 1.6 million);
// 5M-edge graph, 400,000-edge hub graph by BiT-PC: no leaf above 2^20.
bool leaf_part(const SplitJob &c, int depth, uint32_t most) {
    return c.ne < kLeafCap && c.work <= most &&
           (c.work <= kLeafWedges || c.ne < 512 || c.stuck || depth > 5);
}

// BT_LEAF_WEDGES_LOG2 (0..25) sets another bound, for tests and measurements.
uint32_t leaf_most() {
    const char *v = std::getenv("BT_LEAF_WEDGES_LOG2");
    const int l = v ? std::atoi(v) : -1;
    return uint32_t(1) << (l >= 0 && l <= 25 ? l : kLeafMostLog2);
}

// Workspace names of one of the two sets.
struct Names {
    char buf[32];
    const char *operator()(const char *base, int depth) {
        std::snprintf(buf, sizeof buf, "%s%d", base, depth & 1);
        return buf;
    }
};

}  // namespace

void regroup(const SplitIndex &ix, const SweepResult &sw, const std::vector<SplitJob> &jobs,
             int depth, int64_t *phi_out, std::vector<int32_t> &levels, int32_t &max_level,
             Regrouped &out, LeafPool &pool, Workspace &ws, hipStream_t s) {
    Names nm;
    const int64_t m = ix.m, nw = ix.n_w;
    const int32_t np = sw.n_parts;
    out.jobs.clear();
    std::vector<SplitJob> leaves;
    const uint32_t most = leaf_most();
    // Edges by part.
    uint64_t *ekeys = ws.get<uint64_t>("rg_ekeys", m);
    uint32_t *evals = ws.get<uint32_t>("rg_evals", m);
    int64_t *first = ws.get<int64_t>("rg_bounds", 2 * ((int64_t)np + 1));
    int64_t *last = first + np + 1;
    zero_bytes(first, sizeof(int64_t) * 2 * ((size_t)np + 1), s);
    k_edge_keys<<<grid_for(m, 256, 16384), 256, 0, s>>>(sw.mark, m, np, ekeys, evals);
    BT_CHECK_LAUNCH();
    radix_sort_u64_u32(ekeys, evals, m, bits_for((uint64_t)np), ws, s);
    k_part_bounds<<<grid_for(m, 256, 16384), 256, 0, s>>>(ekeys, m, first, last);
    BT_CHECK_LAUNCH();
    int32_t *wpart = ws.get<int32_t>("rg_wpart", nw);
    uint32_t *wcount = ws.get<uint32_t>("rg_wcount", (int64_t)np + 1);
    zero_bytes(wcount, sizeof(uint32_t) * ((size_t)np + 1), s);
    if (nw > 0) {
        if (np < kLdsParts)
            k_wedge_parts<true><<<grid_for(nw, 1024, 512), 1024, sizeof(uint32_t) * (np + 1), s>>>(
                ix.wea, ix.web, nw, sw.mark, np, wpart, wcount);
        else
            k_wedge_parts<false><<<grid_for(nw, 1024, 2048), 1024, 0, s>>>(
                ix.wea, ix.web, nw, sw.mark, np, wpart, wcount);
        BT_CHECK_LAUNCH();
    }
    std::vector<uint32_t> wcnt((size_t)np + 1);
    BT_HIP(hipMemcpyAsync(wcnt.data(), wcount, sizeof(uint32_t) * wcnt.size(),
                          hipMemcpyDeviceToHost, s));
    std::vector<SplitPart> parts((size_t)np);
    std::vector<int64_t> bounds(2 * ((size_t)np + 1));
    BT_HIP(hipMemcpyAsync(parts.data(), sw.parts, sizeof(SplitPart) * np, hipMemcpyDeviceToHost, s));
    BT_HIP(hipMemcpyAsync(bounds.data(), first, sizeof(int64_t) * bounds.size(),
                          hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    // Parts of one level are done; of the others, those that fit one
    // workgroup are leaves and the rest jobs of the next depth.
    int64_t sorted = 0;  // edges that lie in some part
    for (int32_t p = 0; p < np; ++p) {
        const int64_t n = bounds[(size_t)np + 1 + p] - bounds[(size_t)p];
        sorted += n;
        if (n == 0) continue;
        const SplitPart &P = parts[(size_t)p];
        const SplitJob &J = jobs[(size_t)P.job];
        if (P.lo >= P.hi || P.pad) {
            levels[(size_t)J.root] += 1;
            max_level = std::max(max_level, P.hi);
            continue;
        }
        SplitJob c;
        c.part = p;
        c.e0 = 0;
        c.ne = (int32_t)n;
        c.root = J.root;
        c.hi = std::min(P.hi, J.hi);
        c.stuck = n == J.ne;
        c.work = wcnt[(size_t)p];
        (leaf_part(c, depth, most) ? leaves : out.jobs).push_back(c);
    }
    const int32_t nj = (int32_t)out.jobs.size(), nl = (int32_t)leaves.size();
    const uint32_t n_ranks = (uint32_t)(nj + nl);
    std::vector<PartMap> map((size_t)np + 1);
    for (int32_t p = 0; p < np; ++p) map[(size_t)p] = PartMap{~parts[(size_t)p].hi, 0xffffffffu};
    map[(size_t)np] = PartMap{~0, 0xffffffffu};
    for (int32_t j = 0; j < nj + nl; ++j) {
        SplitJob &c = j < nj ? out.jobs[(size_t)j] : leaves[(size_t)(j - nj)];
        int64_t &at = j < nj ? out.m : pool.m;
        c.e0 = (int32_t)at;
        at += c.ne;
        map[(size_t)c.part] = PartMap{c.e0, (uint32_t)j};
    }
    PartMap *dmap = ws.get<PartMap>("rg_map", (int64_t)np + 1);
    BT_HIP(hipMemcpyAsync(dmap, map.data(), sizeof(PartMap) * map.size(), hipMemcpyHostToDevice, s));
    int32_t *newid = ws.get<int32_t>("rg_newid", m);
    out.oid = ws.get<int32_t>(nm("rg_oid", depth), out.m);
    k_renumber<<<grid_for(sorted, 256, 16384), 256, 0, s>>>(ekeys, evals, sorted, dmap, first,
                                                            ix.oid, newid, (uint32_t)nj, out.oid,
                                                            pool.oid, phi_out);
    BT_CHECK_LAUNCH();
    // Wedges: count the kept ones, compact them in bloom order, sort by rank.
    const int64_t tiles = ceil_div(nw, kTile);
    int32_t *tile = ws.get<int32_t>("rg_tile", tiles + 1);
    int64_t *toff = ws.get<int64_t>("rg_tile_off", tiles + 2);
    int64_t *h = ws.host(4);
    h[0] = 0;
    if (n_ranks > 0 && nw > 0) {
        k_keep_count<<<grid_for(tiles, 1, 16384), 256, 0, s>>>(wpart, nw, dmap, n_ranks, tile);
        BT_CHECK_LAUNCH();
        scan_exclusive_i32_to_i64(tile, toff, tiles, ws, s);
        BT_HIP(hipMemcpyAsync(h, toff + tiles, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    }
    BT_HIP(hipStreamSynchronize(s));  // `map` is read until here
    const int64_t n = h[0];
    std::vector<int64_t> rb(2 * ((size_t)nl + 1), 0);
    // The sort's arrays share the memory of the next depth's links.
    uint64_t *keys = reinterpret_cast<uint64_t *>(ws.get<uint3>("sp_link", n + 2));
    uint32_t *vals = reinterpret_cast<uint32_t *>(keys + n + 1);
    if (n > 0) {
        k_keep_write<<<grid_for(tiles, 1, 16384), 256, 0, s>>>(wpart, ix.wbl, nw, dmap, n_ranks,
                                                               toff, keys, vals);
        BT_CHECK_LAUNCH();
        radix_sort_u64_u32(keys, vals, n, bits_for((uint64_t)n_ranks - 1), ws, s);
        const int64_t t2 = ceil_div(n, kTile);
        k_head_count<<<grid_for(t2, 1, 16384), 256, 0, s>>>(keys, n, tile);
        BT_CHECK_LAUNCH();
        scan_exclusive_i32_to_i64(tile, toff, t2, ws, s);  // toff[t2]: all heads
        int64_t *db = ws.get<int64_t>("rg_rank_bounds", 2 * ((int64_t)nl + 1));
        k_rank_bounds<<<grid_for(nl + 1, 4, 1024), 256, 0, s>>>(keys, n, toff, nj, nj + nl, db);
        BT_CHECK_LAUNCH();
        BT_HIP(hipMemcpyAsync(rb.data(), db, sizeof(int64_t) * rb.size(), hipMemcpyDeviceToHost, s));
        BT_HIP(hipStreamSynchronize(s));
    }
    const int64_t n_b = rb[2 * (size_t)nl + 1];
    out.n_w = rb[0];
    out.n_b = rb[1];
    out.wea = ws.get<int32_t>(nm("rg_wea", depth), out.n_w + 1);
    out.web = ws.get<int32_t>(nm("rg_web", depth), out.n_w + 1);
    out.wbl = ws.get<int32_t>(nm("rg_wbl", depth), out.n_w);
    out.bwoff = ws.get<uint32_t>(nm("rg_bwoff", depth), out.n_b + 1);
    out.bk = ws.get<int32_t>(nm("rg_bk", depth), out.n_b + 1);
    zero_bytes(out.bk, sizeof(int32_t) * (out.n_b + 1), s);
    const int64_t lb = n_b - out.n_b, lw = n - out.n_w;
    if (lb > 0) zero_bytes(pool.bk + pool.n_b, sizeof(int32_t) * lb, s);
    if (n > 0) {
        const Dest J{out.wea, out.web, out.wbl, out.bk, out.bwoff, 0, 0};
        const Dest L{pool.wea, pool.web, pool.wbl, pool.bk, pool.bwoff, pool.n_w - out.n_w,
                     pool.n_b - out.n_b};
        k_build<<<grid_for(ceil_div(n, kTile), 1, 16384), 256, 0, s>>>(
            keys, vals, n, out.n_w, toff, ix.wea, ix.web, sw.wedge_k, sw.mark, dmap, newid, J, L);
        BT_CHECK_LAUNCH();
    }
    // Each array's last bloom ends where its wedges do; the next depth's
    // blooms of the pool overwrite that word with the same value.
    k_put_u32<<<1, 1, 0, s>>>(out.bwoff + out.n_b, (uint32_t)out.n_w);
    BT_CHECK_LAUNCH();
    k_put_u32<<<1, 1, 0, s>>>(pool.bwoff + pool.n_b + lb, (uint32_t)(pool.n_w + lw));
    BT_CHECK_LAUNCH();
    for (int32_t j = 0; j < nl; ++j) {
        const SplitJob &c = leaves[(size_t)j];
        LeafJob L;
        L.e0 = c.e0;
        L.ne = c.ne;
        L.w0 = (uint32_t)(pool.n_w + rb[2 * (size_t)j] - out.n_w);
        L.nw = (uint32_t)(rb[2 * (size_t)j + 2] - rb[2 * (size_t)j]);
        L.b0 = (uint32_t)(pool.n_b + rb[2 * (size_t)j + 1] - out.n_b);
        L.nb = (uint32_t)(rb[2 * (size_t)j + 3] - rb[2 * (size_t)j + 1]);
        L.graph = c.root;
        L.id = (int32_t)pool.jobs.size();
        pool.jobs.push_back(L);
        pool.leaves.push_back(c);
    }
    pool.n_w += lw;
    pool.n_b += lb;
}

void LeafPool::place(const void *mem, int64_t nw, int64_t edges, Workspace &ws) {
    int32_t *at = (int32_t *)mem;
    const auto take = [&](int64_t n) {
        int32_t *p = at;
        at += n;
        return p;
    };
    wea = take(nw);
    web = take(nw);
    wbl = take(nw);
    bk = take(nw + 1);
    bwoff = (uint32_t *)take(nw + 1);
    oid = ws.get<int32_t>("pool_oid", edges);
}

void regroup_links(const Regrouped &g, uint64_t *supl, int64_t *link_off, uint3 *link,
                   Workspace &ws, hipStream_t s) {
    const int64_t m = g.m, nw = g.n_w;
    zero_bytes(supl, sizeof(uint64_t) * (m + 1), s);
    if (nw > 0) {
        k_job_supports<<<grid_for(nw, 256, 65536), 256, 0, s>>>(g.wea, g.web, g.wbl, g.bk, nw,
                                                               (unsigned long long *)supl);
        BT_CHECK_LAUNCH();
    }
    int32_t *cnt = ws.get<int32_t>("rg_cnt", m);
    k_job_link_counts<<<grid_for(m, 256, 16384), 256, 0, s>>>(supl, m, cnt);
    BT_CHECK_LAUNCH();
    scan_exclusive_i32_to_i64(cnt, link_off, m, ws, s);
    if (nw > 0) {
        k_job_links<<<grid_for(nw, 256, 65536), 256, 0, s>>>(
            g.wea, g.web, g.wbl, nw, (unsigned long long *)supl, link_off, link);
        BT_CHECK_LAUNCH();
    }
}

}  // namespace bt
