// graph.hip - input validation, vertex priority order and the rank-space
// adjacency (priority of Definition 6; the "p(v) < p(u)" filters of
// Algorithm 3's sweeps become row prefixes).
#include <algorithm>

#include "pipeline.h"

namespace bt {

namespace {

constexpr int kBlock = 256;

// Largest row r in [lo, hi] with row_ptr[r] <= e (lo if there is none).
__device__ __forceinline__ int32_t upper_row_of(const int64_t *row_ptr, int32_t lo, int32_t hi,
                                                int64_t e) {
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo + 1) / 2;
        if (row_ptr[mid] <= e) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Validation flags.
enum : int32_t {
    kBadRowPtr = 1,   // row_ptr not a partition of [0, m)
    kBadCol = 2,      // lower id out of range
    kUnsorted = 4,    // lower ids not strictly increasing in a row (or duplicate)
};

// One thread a row, then one an edge (a wave a row takes 2 ms where one of
// 20M edges' rows holds 165,000).  Where lower ids do not increase a row has
// to begin, which is looked up; with bad row bounds the answer is arbitrary
// but the search stays inside row_ptr, and the bounds are reported first.
__global__ __launch_bounds__(kBlock) void k_validate(const int64_t *row_ptr, const int32_t *col,
                                                     int32_t n_upper, int32_t n_lower,
                                                     int64_t m, int32_t *flags) {
    const int64_t t0 = blockIdx.x * (int64_t)kBlock + threadIdx.x, nt = (int64_t)gridDim.x * kBlock;
    int32_t bad = 0;
    for (int64_t i = t0; i < n_upper; i += nt) {
        const int64_t a = row_ptr[i], b = row_ptr[i + 1];
        if (i == 0 && a != 0) bad |= kBadRowPtr;
        if (i == n_upper - 1 && b != m) bad |= kBadRowPtr;
        if (a < 0 || b < a || b > m) bad |= kBadRowPtr;
    }
    for (int64_t k = t0; k < m; k += nt) {
        const int32_t c = col[k];
        if (c < 0 || c >= n_lower) bad |= kBadCol;
        if (k + 1 < m && col[k + 1] <= c &&
            row_ptr[upper_row_of(row_ptr, 0, n_upper - 1, k + 1)] != k + 1)
            bad |= kUnsorted;
    }
    bad = wave_or(bad);
    if (lane_id() == 0 && bad) atomicOr(flags, bad);
}

// deg[gid]: lower j -> j, upper i -> n_lower + i.  Lower degrees start at zero.
__global__ void k_degrees(const int64_t *row_ptr, const int32_t *col, int64_t m, int32_t n_upper,
                          int32_t n_lower, int32_t *deg) {
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = t0; i < n_upper; i += nt)
        deg[n_lower + i] = (int32_t)(row_ptr[i + 1] - row_ptr[i]);
    for (int64_t e = t0; e < m; e += nt) atomicAdd(&deg[col[e]], 1);
}

__global__ void k_lower_degree(const int32_t *col, int64_t m, int32_t *deg) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&deg[col[e]], 1);
}

// Sort key: layer above degree; the stable sort keeps id order on ties.
__global__ void k_rank_keys(const int32_t *deg, int32_t n_lower, int32_t n, int dbits,
                            uint64_t *keys, uint32_t *vals) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        keys[v] = ((uint64_t)(v >= n_lower) << dbits) | (uint64_t)deg[v];
        vals[v] = (uint32_t)v;
    }
}

// Graph of vertex v in a union (offsets of its layer, n + 1 entries).
__device__ __forceinline__ int32_t comp_of(const int64_t *off, int32_t n, int64_t local) {
    int32_t lo = 0, hi = n - 1;  // largest c with off[c] <= local
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) / 2;
        if (off[mid] <= local) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Union: layer above graph above degree; the stable sort keeps id order.
__global__ void k_rank_keys_comp(const int32_t *deg, int32_t n_lower, int32_t n, Components cp,
                                 int cbits, int dbits, uint64_t *keys, uint32_t *vals) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        const bool up = v >= n_lower;
        const int32_t c = up ? comp_of(cp.u_off, cp.n, v - n_lower) : comp_of(cp.l_off, cp.n, v);
        keys[v] = ((uint64_t)up << (dbits + cbits)) | ((uint64_t)c << dbits) | (uint64_t)deg[v];
        vals[v] = (uint32_t)v;
    }
}

// zbase[p]: the first rank of p's graph in p's layer; vgraph[p]: the graph.
__global__ void k_zbase(const int32_t *new2old, int32_t n_lower, int32_t n, Components cp,
                        int32_t *zbase, int32_t *vgraph) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = new2old[p];
        const bool up = v >= n_lower;
        const int32_t c = up ? comp_of(cp.u_off, cp.n, v - n_lower) : comp_of(cp.l_off, cp.n, v);
        zbase[p] = up ? n_lower + (int32_t)cp.u_off[c] : (int32_t)cp.l_off[c];
        vgraph[p] = c;
    }
}

__global__ void k_rank_apply(const uint32_t *order, const int32_t *deg, int32_t n,
                             int32_t *old2new, int32_t *new2old, int32_t *deg_new) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = (int32_t)order[p];
        old2new[v] = (int32_t)p;
        new2old[p] = v;
        deg_new[p] = deg[v];
    }
}

// The edges in upper rank order: key (upper rank in its layer << nbl | lower
// rank), value the edge.  A wave takes runs of edges, whatever their rows.
__global__ __launch_bounds__(kBlock) void k_entries(const int64_t *row_ptr, const int32_t *col,
                                                    int64_t m, int32_t n_upper, int32_t n_lower,
                                                    const int32_t *old2new, const int64_t *off,
                                                    int nbl, int run_len, uint64_t *keys, uint32_t *vals) {
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t run = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; run * run_len < m;
         run += waves) {
        const int64_t e0 = run * run_len, e1 = min(e0 + run_len, m);
        const int32_t first = upper_row_of(row_ptr, 0, n_upper - 1, e0);
        const int32_t last = upper_row_of(row_ptr, first, n_upper - 1, e1 - 1);
        for (int64_t e = e0 + lane_id(); e < e1; e += kWave) {
            const int32_t i = upper_row_of(row_ptr, first, last, e);
            const int32_t ru = old2new[n_lower + i];
            const uint64_t rl = (uint64_t)old2new[col[e]];
            const int64_t at = off[ru] - m + (e - row_ptr[i]);
            keys[at] = ((uint64_t)(ru - n_lower) << nbl) | rl;
            vals[at] = (uint32_t)e;
        }
    }
}

// Rows of one layer from the sorted edges: adj and eid, and the row's vertex.
__global__ void k_entries_apply(const uint64_t *keys, const uint32_t *vals, int64_t m, int nbl,
                                int32_t n_lower, bool upper, int32_t *adj, int32_t *eid,
                                int32_t *src) {
    const uint64_t mask = (uint64_t(1) << nbl) - 1;
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < m;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int32_t rl = (int32_t)(keys[j] & mask), ru = n_lower + (int32_t)(keys[j] >> nbl);
        adj[j] = upper ? rl : ru;
        src[j] = upper ? ru : rl;
        eid[j] = (int32_t)vals[j];
    }
}

__device__ __forceinline__ uint64_t prio(const int32_t *deg_new, const int32_t *new2old,
                                         int32_t v) {
    return ((uint64_t)deg_new[v] << 31) | (uint64_t)new2old[v];
}

// low[x] = number of neighbours of lower priority (a prefix of the row).
__global__ void k_low(const int64_t *off, const int32_t *adj, const int32_t *deg_new,
                      const int32_t *new2old, int32_t n, int32_t *low) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n;
         x += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t px = prio(deg_new, new2old, (int32_t)x);
        int64_t lo = off[x], hi = off[x + 1];
        while (lo < hi) {  // first neighbour with priority above x
            const int64_t mid = lo + (hi - lo) / 2;
            if (prio(deg_new, new2old, adj[mid]) < px) lo = mid + 1;
            else hi = mid;
        }
        low[x] = (int32_t)(lo - off[x]);
    }
}

// rev for prefix entries (x -> y): position of x in row y.  zlen (nullable)
// for all entries: the entries of row y above both x and y, and rst.
__global__ void k_rev(const int32_t *src, int64_t n2, const int64_t *off, const int32_t *adj,
                      const int32_t *low, int32_t *rev, int32_t *zlen,
                      uint32_t *rst) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n2;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = src[j];
        int32_t r = 0;
        const int32_t y = adj[j];
        const bool down = j - off[x] < low[x];
        if (!down) {
            if (zlen) {
                zlen[j] = (int32_t)(off[y + 1] - off[y]) - low[y];
                rst[j] = (uint32_t)off[y] + low[y];
            }
        } else {
            int64_t lo = off[y], hi = off[y + 1];
            while (lo < hi) {
                const int64_t mid = lo + (hi - lo) / 2;
                if (adj[mid] < x) lo = mid + 1;
                else hi = mid;
            }
            r = (int32_t)(lo - off[y]);
            if (zlen) {
                zlen[j] = (int32_t)(off[y + 1] - lo) - 1;
                rst[j] = (uint32_t)off[y];
            }
        }
        rev[j] = r;
    }
}

}  // namespace

void validate_graph(const bt_csr &g, Workspace &ws, hipStream_t s) {
    const int32_t nu = g.n_upper, nl = g.n_lower;
    const int64_t m = g.m;
    int64_t *hs = ws.host(4);
    int32_t *flags = ws.get<int32_t>("prep_flags", 4);
    zero_bytes(flags, 4 * sizeof(int32_t), s);
    if (nu > 0) {
        k_validate<<<grid_for(std::max<int64_t>(nu, m), kBlock, 4096), kBlock, 0, s>>>(
            g.row_ptr, g.col, nu, nl, m, flags);
        BT_CHECK_LAUNCH();
    }
    BT_HIP(hipMemcpyAsync(hs, flags, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    const int32_t f = *(int32_t *)hs;
    if (nu == 0 && m != 0) throw Error{BT_EINVAL, "graph has edges but no upper vertices"};
    if (f & kBadRowPtr) throw Error{BT_EINVAL, "row_ptr is not a partition of [0, m)"};
    if (f & kBadCol) throw Error{BT_EINVAL, "a lower id is out of range"};
    if (f & kUnsorted)
        throw Error{BT_EINVAL, "lower ids not strictly increasing within a row (duplicate edge?)"};
}

// The priority order of up to kRankSmall vertices of one graph by one
// workgroup: what k_rank_keys, the sort, k_rank_apply and the scan of the
// degrees do in seven launches, each of which costs more than its work (2,500
// vertices: 12 us, before about 45 with the gaps between them; with two scans
// in one launch and sorts that leave their result where the last pass wrote it,
// the 10,000-edge graph's support count 190 -> 157 us).  LDS holds (layer, degree, id) in one word; two stable
// counting passes over layer and degree, in which each wave ranks its own run
// of rows by ballots.
constexpr int kRankBlock = 1024;
constexpr int32_t kRankSmall = 1 << 13;
constexpr int kRankIdBits = 13, kRankDigit = 8;

__global__ __launch_bounds__(kRankBlock) void k_rank_small(const int32_t *deg, int32_t n_lower,
                                                           int32_t n, int dbits, int32_t *old2new,
                                                           int32_t *new2old, int32_t *deg_new,
                                                           int64_t *off) {
    constexpr int kWaves = kRankBlock / kWave;
    __shared__ uint32_t s_key[2][kRankSmall];
    __shared__ uint32_t s_cnt[kWaves << kRankDigit];  // [wave][digit]
    __shared__ uint32_t s_scr[kWaves + 1];
    __shared__ int64_t s_scr64[kWaves + 1];
    const int w = threadIdx.x / kWave;
    const int32_t rows = (n + kRankBlock - 1) / kRankBlock;  // of a wave
    for (int32_t v = threadIdx.x; v < n; v += kRankBlock)
        s_key[0][v] = ((((uint32_t)(v >= n_lower) << dbits) | (uint32_t)deg[v]) << kRankIdBits) |
                      (uint32_t)v;
    uint32_t *const mine = s_cnt + (w << kRankDigit);
    for (int pass = 0, done = 0; pass < 2; ++pass) {
        const uint32_t *in = s_key[pass];
        uint32_t *out = s_key[pass ^ 1];
        const int bits = pass == 0 ? (dbits + 2) / 2 : dbits + 1 - done;
        const int shift = kRankIdBits + done, bins = 1 << bits;
        for (int i = threadIdx.x; i < kWaves << kRankDigit; i += kRankBlock) s_cnt[i] = 0;
        __syncthreads();
        for (int32_t i = 0; i < rows; ++i) {
            const int32_t x = (w * rows + i) * kWave + lane_id();
            if (x < n) atomicAdd(&mine[(in[x] >> shift) & (uint32_t)(bins - 1)], 1u);
        }
        __syncthreads();
        uint32_t sum = 0, all;
        if ((int)threadIdx.x < bins)
            for (int j = 0; j < kWaves; ++j) sum += s_cnt[(j << kRankDigit) + threadIdx.x];
        uint32_t pos = block_exclusive_sum<uint32_t>(sum, s_scr, &all);
        if ((int)threadIdx.x < bins)
            for (int j = 0; j < kWaves; ++j) {
                const uint32_t c = s_cnt[(j << kRankDigit) + threadIdx.x];
                s_cnt[(j << kRankDigit) + threadIdx.x] = pos;
                pos += c;
            }
        __syncthreads();
        for (int32_t i = 0; i < rows; ++i) {
            const int32_t x = (w * rows + i) * kWave + lane_id();
            const bool ok = x < n;
            const uint32_t k = ok ? in[x] : 0u;
            const uint32_t d = (k >> shift) & (uint32_t)(bins - 1);
            uint64_t peers = __ballot(ok);
            for (int b = 0; b < bits; ++b) {
                const bool bit = (d >> b) & 1;
                const uint64_t bal = __ballot(bit);
                peers &= bit ? bal : ~bal;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t at = mine[d] + rank;
            if (ok) out[at] = k;
            wave_fence();  // all lanes have read the position
            if (ok && rank == 0) mine[d] = at + (uint32_t)__popcll(peers);
            wave_fence();
        }
        __syncthreads();
        done += bits;
    }
    // Back in s_key[0].  Each thread takes a run of ranks.
    const int32_t p0 = (int32_t)threadIdx.x * rows;
    int64_t sum = 0, all;
    const uint32_t dmask = (1u << dbits) - 1;
    for (int32_t p = p0; p < min(p0 + rows, n); ++p) sum += (s_key[0][p] >> kRankIdBits) & dmask;
    int64_t run = block_exclusive_sum<int64_t>(sum, s_scr64, &all);
    for (int32_t p = p0; p < min(p0 + rows, n); ++p) {
        off[p] = run;
        run += (s_key[0][p] >> kRankIdBits) & dmask;
    }
    if (threadIdx.x == 0) off[n] = all;
    for (int32_t p = threadIdx.x; p < n; p += kRankBlock) {
        const uint32_t k = s_key[0][p];
        const int32_t v = (int32_t)(k & ((1u << kRankIdBits) - 1));
        old2new[v] = p;
        new2old[p] = v;
        deg_new[p] = (int32_t)((k >> kRankIdBits) & dmask);
    }
}

void prepare(const bt_csr &g, RankCSR &r, Workspace &ws, hipStream_t s,
             const Components *comps, bool up) {
    const int32_t nu = g.n_upper, nl = g.n_lower;
    const int64_t m = g.m;
    const int64_t n = (int64_t)nu + nl;
    r.tp = tune_params(false, m);
    r.n_lower = nl;
    r.n = (int32_t)n;
    r.m = m;

    validate_graph(g, ws, s);

    // Degrees and the priority order.
    int32_t *deg = ws.get<int32_t>("prep_deg", n);
    zero_bytes(deg, sizeof(int32_t) * (nl > 0 ? nl : 1), s);
    if (n > 0) {
        k_degrees<<<grid_for(std::max<int64_t>(nu, m), 256, 16384), 256, 0, s>>>(
            g.row_ptr, g.col, m, nu, nl, deg);
        BT_CHECK_LAUNCH();
    }
    int32_t *old2new = ws.get<int32_t>("prep_old2new", n);
    int32_t *new2old = ws.get<int32_t>("prep_new2old", n);
    int32_t *deg_new = ws.get<int32_t>("prep_degnew", n);
    const bool uni = comps && comps->n > 1;
    r.zbase = r.vgraph = nullptr;
    // No degree exceeds the size of the other layer.
    const int dbits = bits_for((uint64_t)std::max(nu, nl));
    r.off = ws.get<int64_t>("rank_off", n + 1);
    const bool small = !uni && n > 0 && n <= kRankSmall;
    if (small) {
        k_rank_small<<<1, kRankBlock, 0, s>>>(deg, nl, (int32_t)n, dbits, old2new, new2old, deg_new,
                                              r.off);
        BT_CHECK_LAUNCH();
    } else if (n > 0) {
        uint64_t *vkeys = ws.get<uint64_t>("prep_vkeys", n);
        uint32_t *vorder = ws.get<uint32_t>("prep_vorder", n);
        if (uni) {
            const int cbits = bits_for((uint64_t)(comps->n - 1));
            k_rank_keys_comp<<<grid_for(n, 256, 8192), 256, 0, s>>>(deg, nl, (int32_t)n, *comps,
                                                                   cbits, dbits, vkeys, vorder);
            BT_CHECK_LAUNCH();
            radix_sort_u64_u32(vkeys, vorder, n, dbits + cbits + 1, ws, s);
        } else {
            k_rank_keys<<<grid_for(n, 256, 8192), 256, 0, s>>>(deg, nl, (int32_t)n, dbits, vkeys,
                                                              vorder);
            BT_CHECK_LAUNCH();
            radix_sort_u64_u32(vkeys, vorder, n, dbits + 1, ws, s);
        }
        k_rank_apply<<<grid_for(n, 256, 8192), 256, 0, s>>>(vorder, deg, (int32_t)n, old2new,
                                                            new2old, deg_new);
        BT_CHECK_LAUNCH();
        if (uni) {
            r.zbase = ws.get<int32_t>("rank_zbase", n);
            r.vgraph = ws.get<int32_t>("rank_vgraph", n);
            k_zbase<<<grid_for(n, 256, 8192), 256, 0, s>>>(new2old, nl, (int32_t)n, *comps,
                                                           r.zbase, r.vgraph);
            BT_CHECK_LAUNCH();
        }
    }
    if (!small) scan_exclusive_i32_to_i64(deg_new, r.off, n, ws, s);

    // Rank-space rows sorted by neighbour priority: the edges in upper rank
    // order, sorted (stably) by lower rank, are the lower rows; those, sorted
    // by upper rank, are the upper rows.
    const int64_t n2 = 2 * m;
    const int nbl = bits_for((uint64_t)std::max(nl - 1, 0)), nbu = bits_for((uint64_t)std::max(nu - 1, 0));
    uint64_t *ekeys = ws.get<uint64_t>("prep_ekeys", m);
    uint32_t *evals = ws.get<uint32_t>("prep_evals", m);
    int32_t *src = ws.get<int32_t>("prep_src", n2);
    r.adj = ws.get<int32_t>("rank_adj", n2);
    r.eid = ws.get<int32_t>("rank_eid", n2);
    r.rev = ws.get<int32_t>("rank_rev", n2);
    r.low = ws.get<int32_t>("rank_low", n);
    r.wpre = ws.get<int64_t>("rank_wpre", n2 + 1);
    r.zlen = up ? ws.get<int32_t>("rank_zlen", n2) : nullptr;
    r.rst = up ? ws.get<uint32_t>("rank_rst", n2) : nullptr;
    r.zpre = up ? ws.get<int64_t>("rank_zpre", n2 + 1) : nullptr;
    if (m > 0) {
        // Short runs where there are too few to fill the chip.
        const int run = m < (int64_t(1) << 20) ? kWave : 8 * kWave;
        k_entries<<<grid_for(ceil_div(m, run) * kWave, kBlock, 8192), kBlock, 0, s>>>(
            g.row_ptr, g.col, m, nu, nl, old2new, r.off, nbl, run, ekeys, evals);
        BT_CHECK_LAUNCH();
        uint64_t *ekeys2 = ws.get<uint64_t>("rs_keys", m);
        uint32_t *evals2 = ws.get<uint32_t>("rs_vals", m);
        for (const bool upper : {false, true}) {
            radix_sort_swap(ekeys, evals, ekeys2, evals2, m, upper ? nbu : nbl, ws, s,
                            upper ? nbl : 0);
            k_entries_apply<<<grid_for(m, 256, 16384), 256, 0, s>>>(
                ekeys, evals, m, nbl, nl, upper, r.adj + (upper ? m : 0), r.eid + (upper ? m : 0),
                src + (upper ? m : 0));
            BT_CHECK_LAUNCH();
        }
    }
    if (n > 0) {
        k_low<<<grid_for(n, 256, 8192), 256, 0, s>>>(r.off, r.adj, deg_new, new2old,
                                                     (int32_t)n, r.low);
        BT_CHECK_LAUNCH();
    }
    if (m > 0) {
        k_rev<<<grid_for(n2, 256, 16384), 256, 0, s>>>(src, n2, r.off, r.adj, r.low,
                                                       r.rev, r.zlen, r.rst);
        BT_CHECK_LAUNCH();
    }
    if (up) scan_two_i32_to_i64(r.rev, r.wpre, r.zlen, r.zpre, n2, ws, s);
    else scan_exclusive_i32_to_i64(r.rev, r.wpre, n2, ws, s);
}

// ------------------------------------------------------------- tasks

namespace {

__device__ __forceinline__ int64_t vertex_work(const int64_t *off, const int32_t *low,
                                               const int64_t *wpre, int32_t x) {
    return wpre[off[x] + low[x]] - wpre[off[x]];
}

// Start vertices with more than hash_max wedges count their end vertices
// in ranges of the ranks below x in x's layer (in a union, x's graph's part of
// it), one task per range: of `chunk` ids, one dense counter each, or, where
// those would hold few wedges, shares of the degrees with half of hash_max
// wedges each on average, which a hash table takes.  A start of 10,000 wedges
// over 500,000 ids had 81 dense ranges; the heavy starts of the 5M-edge graph
// took 18.5 ms with dense ranges alone and 14.8 ms so.
__device__ __forceinline__ int32_t z_base(const int32_t *zbase, int32_t x, int32_t n_lower) {
    return zbase ? zbase[x] : (x >= n_lower ? n_lower : 0);
}
__device__ __forceinline__ int32_t dense_chunks(int32_t x, int32_t base, int32_t chunk) {
    return (x - base + chunk - 1) / chunk;
}
// Tasks of a heavy start: dense ranges, or shares (negative).
__device__ __forceinline__ int32_t heavy_tasks(int32_t x, int32_t base, int32_t chunk, int64_t work,
                                               int32_t hash_max) {
    const int32_t dense = dense_chunks(x, base, chunk);
    const int64_t half = hash_max > 1 ? hash_max / 2 : 1;
    const int64_t shares = (work + half - 1) / half;
    return shares < dense ? -(int32_t)shares : dense;
}

__global__ void k_task_count(const int64_t *off, const int32_t *low, const int64_t *wpre,
                             const int32_t *zbase, int32_t n, int32_t n_lower, int32_t hash_max,
                             int32_t chunk, int64_t *counts) {
    int64_t nh = 0, nd = 0;
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t w = vertex_work(off, low, wpre, (int32_t)x);
        if (w == 0) continue;
        if (w <= hash_max) ++nh;
        else
            nd += abs(heavy_tasks((int32_t)x, z_base(zbase, (int32_t)x, n_lower), chunk, w, hash_max));
    }
    nh = wave_sum(nh);
    nd = wave_sum(nd);
    if (lane_id() == 0) {
        if (nh) atomicAdd((unsigned long long *)&counts[0], (unsigned long long)nh);
        if (nd) atomicAdd((unsigned long long *)&counts[1], (unsigned long long)nd);
    }
}

__global__ void k_task_fill(const int64_t *off, const int32_t *low, const int64_t *wpre,
                            const int32_t *zbase, int32_t n, int32_t n_lower, int32_t hash_max,
                            int32_t chunk, WedgeTask *hash, WedgeTask *dense,
                            int32_t *cursors) {
    for (int64_t xi = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; xi < n;
         xi += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = (int32_t)xi;
        const int64_t w = vertex_work(off, low, wpre, x);
        if (w == 0) continue;
        if (w <= hash_max) {
            int32_t cap = 128;
            while (cap < 2 * w) cap <<= 1;
            const int32_t p = atomicAdd(&cursors[0], 1);
            hash[p] = WedgeTask{x, 0, 0, cap};
        } else {
            const int32_t base = z_base(zbase, x, n_lower);
            const int32_t ht = heavy_tasks(x, base, chunk, w, hash_max);
            const int32_t nc = abs(ht);
            const int32_t p = atomicAdd(&cursors[1], nc);
            for (int32_t c = 0; c < nc; ++c) {
                if (ht < 0) {
                    dense[p + c] = WedgeTask{x, c, nc, -1};
                    continue;
                }
                const int32_t lo = base + c * chunk;
                const int32_t hi = min(lo + chunk, x);
                dense[p + c] = WedgeTask{x, lo, hi, hi - lo};
            }
        }
    }
}

}  // namespace

void make_tasks(const RankCSR &rc, TaskLists &t, Workspace &ws, hipStream_t s) {
    RankCSR &r = const_cast<RankCSR &>(rc);
    if (!tune_valid(r.tp)) throw Error{BT_EINVAL, "invalid launch parameters"};
    int64_t *counts = ws.get<int64_t>("task_counts", 4);
    zero_bytes(counts, 4 * sizeof(int64_t), s);
    if (r.n > 0) {
        k_task_count<<<grid_for(r.n, 256, 4096), 256, 0, s>>>(
            r.off, r.low, r.wpre, r.zbase, r.n, r.n_lower, r.tp.hash_max_work, r.tp.dense_chunk,
            counts);
        BT_CHECK_LAUNCH();
    }
    int64_t *hs = ws.host(4);
    BT_HIP(hipMemcpyAsync(hs, counts, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipMemcpyAsync(hs + 2, r.wpre + 2 * r.m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    t.n_hash = hs[0];
    t.n_dense = hs[1];
    if (t.n_hash >= INT32_MAX || t.n_dense >= INT32_MAX)
        throw Error{BT_EOVERFLOW, "too many wedge tasks"};
    r.wedges_po = hs[2];
    t.hash = ws.get<WedgeTask>("task_hash", t.n_hash);
    t.dense = ws.get<WedgeTask>("task_dense", t.n_dense);
    int32_t *cur = ws.get<int32_t>("task_cursor", 2);
    zero_bytes(cur, 2 * sizeof(int32_t), s);
    if (r.n > 0 && (t.n_hash + t.n_dense) > 0) {
        k_task_fill<<<grid_for(r.n, 256, 4096), 256, 0, s>>>(
            r.off, r.low, r.wpre, r.zbase, r.n, r.n_lower, r.tp.hash_max_work, r.tp.dense_chunk,
            t.hash, t.dense, cur);
        BT_CHECK_LAUNCH();
    }
}

}  // namespace bt

// ------------------------------------------------------ footprint

namespace bt {

namespace {

// sum over edges of min(d(u), d(v)): one wave per upper row.
__global__ __launch_bounds__(kBlock) void k_min_degree_sum(const int64_t *row_ptr,
                                                           const int32_t *col,
                                                           const int32_t *deg_lower,
                                                           int32_t n_upper,
                                                           unsigned long long *out) {
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    unsigned long long acc = 0;
    for (int64_t i = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; i < n_upper;
         i += waves) {
        const int64_t a = row_ptr[i], b = row_ptr[i + 1];
        const int32_t du = (int32_t)(b - a);
        for (int64_t k = a + lane_id(); k < b; k += kWave) {
            const int32_t dl = deg_lower[col[k]];
            acc += (unsigned long long)(du < dl ? du : dl);
        }
    }
    acc = wave_sum(acc);
    if (lane_id() == 0 && acc) atomicAdd(out, acc);
}

}  // namespace

int64_t footprint_bytes(const bt_csr &g, Workspace &ws, hipStream_t s) {
    const int32_t nu = g.n_upper, nl = g.n_lower;
    const int64_t m = g.m;
    int32_t *flags = ws.get<int32_t>("fp_flags", 4);
    int32_t *deg = ws.get<int32_t>("fp_deg", nl);
    unsigned long long *sum = ws.get<unsigned long long>("fp_sum", 1);
    zero_bytes(flags, 4 * sizeof(int32_t), s);
    if (nu > 0) {
        k_validate<<<grid_for(std::max<int64_t>(nu, m), kBlock, 4096), kBlock, 0, s>>>(
            g.row_ptr, g.col, nu, nl, m, flags);
        BT_CHECK_LAUNCH();
    }
    int64_t *hs = ws.host(4);
    BT_HIP(hipMemcpyAsync(hs, flags, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    if (*(int32_t *)hs != 0 || (nu == 0 && m != 0)) throw Error{BT_EINVAL, "malformed graph"};
    zero_bytes(deg, sizeof(int32_t) * (nl > 0 ? nl : 1), s);
    zero_bytes(sum, sizeof(unsigned long long), s);
    if (m > 0) {
        k_lower_degree<<<grid_for(m, 256, 16384), 256, 0, s>>>(g.col, m, deg);
        BT_CHECK_LAUNCH();
        k_min_degree_sum<<<grid_for((int64_t)nu * kWave, kBlock, 16384), kBlock, 0, s>>>(
            g.row_ptr, g.col, deg, nu, sum);
        BT_CHECK_LAUNCH();
    }
    BT_HIP(hipMemcpyAsync(hs, sum, sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    const int64_t wbound = hs[0];  // priority-obeyed wedges <= this (Lemma 6)
    return 68 * wbound + 250 * m + 40 * ((int64_t)nu + nl) + (int64_t(1) << 20);
}

}  // namespace bt
