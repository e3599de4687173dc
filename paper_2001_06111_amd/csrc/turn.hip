// turn.hip - turns of the peels on the device.
#include <condition_variable>
#include <map>

#include "peel_common.h"

namespace bt {

namespace {

// Turns of the cooperative peels: tickets in asking order, the waiting
// tickets with their weights (edges), those of peels that go beside the
// holder, and the yield word the holder's kernels read.  Never destroyed: it
// outlives static teardown.
struct Gate {
    std::mutex mu;
    std::condition_variable cv;
    uint64_t next = 0;
    bool busy = false;
    int64_t holder_weight = 0;
    std::map<uint64_t, int64_t> waiting, beside;
    int32_t *word = nullptr;  // pinned, coherent: [0] yield request, [1] always 1
    int32_t *dword = nullptr;  // its device address
};

constexpr int64_t kYieldRatio = 8;

Gate &gate() {
    static Gate *g = new Gate();
    return *g;
}

// Some of these tickets before `end` is much lighter than w.
bool lighter(const std::map<uint64_t, int64_t> &tickets, int64_t w, uint64_t end = UINT64_MAX) {
    for (const auto &t : tickets)
        if (t.first < end && t.second * kYieldRatio < w) return true;
    return false;
}

// Under g.mu: raise the yield word when some waiter, or a peel beside the
// holder, is much lighter than it, clear it otherwise.
void update_yield(Gate &g) {
    const bool ask =
        g.busy && (lighter(g.waiting, g.holder_weight) || lighter(g.beside, g.holder_weight));
    if (!g.word) return;
    static const bool verbose = std::getenv("BT_PEEL_VERBOSE") != nullptr;
    if (verbose && (g.word[0] != 0) != ask)
        std::fprintf(stderr, "[peel] yield word %d (holder weight %lld, %zu waiting, %zu beside)\n",
                     ask ? 1 : 0, (long long)g.holder_weight, g.waiting.size(), g.beside.size());
    __atomic_store_n(&g.word[0], ask ? 1 : 0, __ATOMIC_RELEASE);
}

// Under g.mu, with `ticket` in g.waiting: waits for it to be the oldest
// waiter while the device is free, then takes the turn.  With `after_beside`
// also for the much lighter peels beside, as far as they asked before (later
// ones raise the word anew, so the holder gets on in between).
void take_turn(Gate &g, std::unique_lock<std::mutex> &lk, uint64_t ticket, int64_t weight,
               bool after_beside) {
    update_yield(g);
    g.cv.wait(lk, [&] {
        return !g.busy && g.waiting.begin()->first == ticket &&
               !(after_beside && lighter(g.beside, weight, ticket));
    });
    g.waiting.erase(ticket);
    g.busy = true;
    g.holder_weight = weight;
    update_yield(g);
}

}  // namespace

namespace {
thread_local int64_t t_turn_weight = -1;
}  // namespace

void set_turn_weight(int64_t w) { t_turn_weight = w; }

CoopTurn::CoopTurn(int64_t weight, bool barriers) : weight_(t_turn_weight >= 0 ? t_turn_weight : weight) {
    Gate &g = gate();
    std::unique_lock<std::mutex> lk(g.mu);
    if (!g.word) {
        void *h = nullptr, *d = nullptr;
        BT_HIP(hipHostMalloc(&h, 2 * sizeof(int32_t),
                             hipHostMallocMapped | hipHostMallocCoherent));
        BT_HIP(hipHostGetDevicePointer(&d, h, 0));
        g.word = static_cast<int32_t *>(h);
        g.word[0] = 0;
        g.word[1] = 1;
        g.dword = static_cast<int32_t *>(d);
    }
    ticket_ = g.next++;
    held_ = barriers;
    if (barriers) {
        g.waiting[ticket_] = weight_;
        take_turn(g, lk, ticket_, weight_, false);
    } else {
        g.beside[ticket_] = weight_;
        update_yield(g);
    }
}

CoopTurn::~CoopTurn() {
    Gate &g = gate();
    std::lock_guard<std::mutex> lk(g.mu);
    if (held_) {
        g.busy = false;
        g.holder_weight = 0;
    } else {
        g.beside.erase(ticket_);
    }
    update_yield(g);
    g.cv.notify_all();
}

const int32_t *CoopTurn::yield_word(bool force) const { return gate().dword + (force ? 1 : 0); }

void CoopTurn::requeue() {
    Gate &g = gate();
    std::unique_lock<std::mutex> lk(g.mu);
    g.busy = false;
    g.holder_weight = 0;
    ticket_ = g.next++;
    g.waiting[ticket_] = weight_;
    g.cv.notify_all();
    take_turn(g, lk, ticket_, weight_, true);
}

}  // namespace bt
