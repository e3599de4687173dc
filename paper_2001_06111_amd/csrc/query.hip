// query.hip - k-bitruss subgraphs and their connected components.
//
// H_k, the k-bitruss (Definition 4), is the set of edges with phi_e >= k
// (Definition 5); the cohesive groups the paper's applications look for
// (Section I) are its connected components.  Given the bitruss numbers,
// the components come from a lock-free union-find over the vertices that
// H_k's edges join: every root is hooked under a smaller root with one
// compare-and-swap, so parents only decrease and no cycle can form.  Edges
// are then labelled by component, numbered in order of each component's
// smallest edge id, which makes the labelling unique.
#include <climits>

#include "pipeline.h"

namespace bt {

namespace {

constexpr int kB = 256;

template <typename T> __device__ __forceinline__ T ldc(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T> __device__ __forceinline__ void stc(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t find_root(const int32_t *parent, int32_t x) {
    int32_t p = ldc(&parent[x]);
    while (p != x) {
        x = p;
        p = ldc(&parent[x]);
    }
    return x;
}

// find_root while hooks run, halving the path it walks: x's parent becomes
// its grandparent, an ancestor of x, so a concurrent walk or hook sees an
// older or a newer ancestor and nothing else.  Only a root is ever hooked,
// and x is no root when it is written here.
__device__ __forceinline__ int32_t find_root_halving(int32_t *parent, int32_t x) {
    int32_t p = ldc(&parent[x]);
    while (p != x) {
        const int32_t g = ldc(&parent[p]);
        if (g != p) stc(&parent[x], g);
        x = p;
        p = g;
    }
    return x;
}

__global__ void k_cc_init(int32_t *parent, int32_t n) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x)
        parent[v] = (int32_t)v;
}

// Vertex ids: lower j -> j, upper i -> n_lower + i.
__global__ void k_cc_hook(const int64_t *row_ptr, const int32_t *col, int32_t nu, int32_t nl,
                          const int64_t *phi, int64_t k, int32_t *parent) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t i = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; i < nu;
         i += waves) {
        const int32_t u = nl + (int32_t)i;
        for (int64_t e = row_ptr[i] + lane_id(); e < row_ptr[i + 1]; e += kWave) {
            if (phi[e] < k) continue;
            int32_t a = u, b = col[e];
            while (true) {
                a = find_root_halving(parent, a);
                b = find_root_halving(parent, b);
                if (a == b) break;
                if (a < b) {
                    const int32_t t = a;
                    a = b;
                    b = t;
                }
                // Hook the larger root a under b; retry if a stopped being a root.
                if (atomicCAS(&parent[a], a, b) == a) break;
            }
        }
    }
}

// All of a row's edges with phi >= k lie in one component (they share the
// upper vertex), so each of the passes below finds the root once a row.
//
// The smallest edge of each component.  A row's candidate is its first edge
// with phi >= k, and it is offered only where it beats the value now stored:
// the largest component takes nearly every row, and one atomic per edge on
// its single word was 9.2 ms of the 11 ms call on a 1M-edge power-law graph.
__global__ void k_cc_min_edge(const int64_t *row_ptr, int32_t nu, int32_t nl, const int64_t *phi,
                              int64_t k, const int32_t *parent, int32_t *min_edge) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t i = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; i < nu;
         i += waves) {
        const int64_t end = row_ptr[i + 1];
        for (int64_t e0 = row_ptr[i]; e0 < end; e0 += kWave) {
            const int64_t e = e0 + lane_id();
            const unsigned long long in = __ballot(e < end && phi[e < end ? e : e0] >= k);
            if (!in) continue;
            if (lane_id() == 0) {
                const int32_t first = (int32_t)(e0 + __ffsll(in) - 1);
                const int32_t root = find_root(parent, nl + (int32_t)i);
                if (ldc(&min_edge[root]) > first) atomicMin(&min_edge[root], first);
            }
            break;
        }
    }
}

// first[e] = 1 when e is the smallest edge of its component.
__global__ void k_cc_first(const int64_t *row_ptr, int32_t nu, int32_t nl, const int64_t *phi,
                           int64_t k, const int32_t *parent, const int32_t *min_edge,
                           int32_t *first) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t i = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; i < nu;
         i += waves) {
        const int32_t me = min_edge[find_root(parent, nl + (int32_t)i)];
        for (int64_t e = row_ptr[i] + lane_id(); e < row_ptr[i + 1]; e += kWave)
            first[e] = phi[e] >= k && me == (int32_t)e ? 1 : 0;
    }
}

__global__ void k_cc_label(const int64_t *row_ptr, int32_t nu, int32_t nl, const int64_t *phi,
                           int64_t k, const int32_t *parent, const int32_t *min_edge,
                           const int64_t *pos, int32_t *comp) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t i = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; i < nu;
         i += waves) {
        // A row without an edge of the k-bitruss has no smallest edge.
        const int32_t me = min_edge[find_root(parent, nl + (int32_t)i)];
        const int32_t c = me == INT_MAX ? -1 : (int32_t)pos[me];
        for (int64_t e = row_ptr[i] + lane_id(); e < row_ptr[i + 1]; e += kWave)
            comp[e] = phi[e] >= k ? c : -1;
    }
}

}  // namespace

int64_t bitruss_components(const bt_csr &g, const int64_t *phi, int64_t k, int32_t *comp,
                           Workspace &ws, hipStream_t s) {
    const int32_t nu = g.n_upper, nl = g.n_lower;
    const int32_t n = nu + nl;
    const int64_t m = g.m;
    if (m == 0) return 0;
    int32_t *parent = ws.get<int32_t>("q_parent", n);
    int32_t *min_edge = ws.get<int32_t>("q_min_edge", n);
    int32_t *first = ws.get<int32_t>("q_first", m);
    int64_t *pos = ws.get<int64_t>("q_pos", m + 1);
    const int grid_v = grid_for(n, kB, 16384);
    const int grid_r = grid_for((int64_t)nu * kWave, kB, 16384);
    k_cc_init<<<grid_v, kB, 0, s>>>(parent, n);
    BT_CHECK_LAUNCH();
    fill_i32(min_edge, INT_MAX, n, s);
    k_cc_hook<<<grid_r, kB, 0, s>>>(g.row_ptr, g.col, nu, nl, phi, k, parent);
    BT_CHECK_LAUNCH();
    k_cc_min_edge<<<grid_r, kB, 0, s>>>(g.row_ptr, nu, nl, phi, k, parent, min_edge);
    BT_CHECK_LAUNCH();
    k_cc_first<<<grid_r, kB, 0, s>>>(g.row_ptr, nu, nl, phi, k, parent, min_edge, first);
    BT_CHECK_LAUNCH();
    scan_exclusive_i32_to_i64(first, pos, m, ws, s);
    k_cc_label<<<grid_r, kB, 0, s>>>(g.row_ptr, nu, nl, phi, k, parent, min_edge, pos, comp);
    BT_CHECK_LAUNCH();
    int64_t *h = ws.host(2);
    BT_HIP(hipMemcpyAsync(h, pos + m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BT_HIP(hipStreamSynchronize(s));
    return h[0];
}

}  // namespace bt
