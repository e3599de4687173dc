// peel_split.h - the grid-wide peel that splits edge sets into ranges of
// bitruss numbers: state shared by the sweep kernels (peel_split.hip) and the
// regrouping of their results (regroup.hip).
#pragma once

#include <memory>

#include "peel_common.h"

namespace bt {

// A part of a job: the edges a sweep removed while it worked at one level.
// Their bitruss numbers lie in [lo, hi].
struct alignas(16) SplitPart {
    int32_t hi;   // the level the sweep worked at
    int32_t lo;   // the smallest support taken when the part began
    int32_t job;
    int32_t pad;  // 1: done whatever its bounds (below a progressive pass's threshold)
};

// What a sweep knows of an edge: its part (-1 while it remains, INT_MAX if an
// earlier pass fixed it) and the round that removes it (INT_MAX while it
// remains), in one word.
struct alignas(8) EdgeMark {
    u64 v;
};
__host__ __device__ __forceinline__ u64 edge_mark(int32_t part, int32_t round) {
    return ((u64)(uint32_t)part << 32) | (uint32_t)round;
}
__device__ __forceinline__ int32_t mark_part(u64 v) { return (int32_t)(v >> 32); }
__device__ __forceinline__ int32_t mark_round(u64 v) { return (int32_t)(uint32_t)v; }

// One depth of the split: jobs (disjoint edge ranges) and their index.
struct SplitIndex {
    int64_t m = 0, n_b = 0, n_w = 0;
    const uint32_t *bwoff = nullptr;
    int32_t *bk = nullptr;
    const int32_t *wea = nullptr, *web = nullptr, *wbl = nullptr;  // kFixedBit: not of this job
    const int64_t *link_off = nullptr;
    const uint3 *link = nullptr;
    const int32_t *oid = nullptr;  // caller's edge of each edge (null: the same)
};

// A job of the next depth, or a leaf: its part, edges and root graph.
struct SplitJob {
    int32_t part;
    int32_t e0, ne;  // in the next depth's numbering, or the pool's
    int32_t root;
    int32_t hi;      // its bitruss numbers are at most this
    uint32_t work = 0;  // its wedges
    bool stuck;      // its job came back whole: split it by levels
};

// What a sweep leaves for the regrouping.
struct SweepResult {
    const EdgeMark *mark;     // [m]
    const int32_t *wedge_k;   // [n_w] at one of the wedges that each part killed of
                              // each bloom: the bloom's live wedges when the part
                              // began; elsewhere 0
    SplitPart *parts;         // device
    int32_t n_parts;
};

// The next depth's jobs.
struct Regrouped {
    int64_t m = 0, n_w = 0, n_b = 0;
    int32_t *wea = nullptr, *web = nullptr, *wbl = nullptr, *bk = nullptr, *oid = nullptr;
    uint32_t *bwoff = nullptr;
    std::vector<SplitJob> jobs;
};

// The leaves of all depths (edges, wedges and blooms appended as they come).
struct LeafPool {
    int64_t m = 0, n_w = 0, n_b = 0;       // taken so far
    int32_t *wea = nullptr, *web = nullptr, *wbl = nullptr, *bk = nullptr, *oid = nullptr;
    uint32_t *bwoff = nullptr;             // ends of the depths' blooms have a slot of their own
    std::vector<SplitJob> leaves;
    std::vector<LeafJob> jobs;             // w0, nw, b0, nb filled by regroup
    // Room for m edges, n_w wedges and as many blooms, at `mem` (24 bytes a
    // wedge).
    void place(const void *mem, int64_t n_w, int64_t m, Workspace &ws);
};

// Sorts the edges, wedges and blooms of a swept depth by part: parts of one
// level get their numbers in phi_out, leaves go to the pool, the others are
// the next depth's jobs.  depth picks between two sets of buffers, so that a
// depth's arrays outlive the next one's making.
void regroup(const SplitIndex &ix, const SweepResult &sw, const std::vector<SplitJob> &jobs,
             int depth, int64_t *phi_out, std::vector<int32_t> &levels, int32_t &max_level,
             Regrouped &out, LeafPool &pool, Workspace &ws, hipStream_t s);

// Peels the pool's leaves (peel_leaf.hip).  A leaf does not wait for other
// parts, so leaves that a depth finds may start beside the deeper sweeps.
class LeafRun {
  public:
    // For a pool of up to m edges and n_w wedges.  With `turn` (and its yield
    // word) the launches end early to give the device to a much lighter peel.
    LeafRun(const LeafPool &pool, int64_t m, int64_t n_w, int64_t *phi_out, bool unit_updates,
            int32_t n_roots, CoopTurn *turn, const int32_t *yield_word, Workspace &ws,
            hipStream_t s);
    ~LeafRun();  // waits for what was started
    LeafRun(const LeafRun &) = delete;
    LeafRun &operator=(const LeafRun &) = delete;
    // Starts the large ones of the leaves found so far, on a stream of their
    // own and by at most so many workgroups (a compute unit each), unless
    // earlier ones still run.
    void start(int groups);
    // Peels what is left to its end; levels[root] grows by each leaf's.
    void finish(std::vector<int32_t> &levels, int32_t &max_level, PeelCounters &pc);

  private:
    struct State;
    void take();
    const LeafPool &pool_;
    bool unit_;
    int32_t roots_;
    CoopTurn *turn_;
    Workspace &ws_;
    hipStream_t s_;
    std::unique_ptr<State> st_;
};

// Supports, link counts and links of a regrouped depth's jobs.
void regroup_links(const Regrouped &g, uint64_t *supl, int64_t *link_off, uint3 *link,
                   Workspace &ws, hipStream_t s);

}  // namespace bt
