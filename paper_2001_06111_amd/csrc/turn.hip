// turn.hip - turns of the peels on the device.
#include <condition_variable>
#include <map>

#include "peel_common.h"

namespace bt {

namespace {

// Turns of the cooperative peels: tickets in asking order, the waiting
// tickets with their weights (edges), and the yield word the holder's
// kernel reads.  Never destroyed: it outlives static teardown.
struct Gate {
    std::mutex mu;
    std::condition_variable cv;
    uint64_t next = 0;
    bool busy = false;
    bool leaves = false;  // the holder runs kernels without grid barriers only
    int64_t holder_weight = 0;
    std::map<uint64_t, int64_t> waiting;
    int32_t *word = nullptr;  // pinned, coherent: [0] yield request, [1] always 1
    int32_t *dword = nullptr;  // its device address
};

constexpr int64_t kYieldRatio = 8;

Gate &gate() {
    static Gate *g = new Gate();
    return *g;
}

// Under g.mu: raise the yield word when some waiter is much lighter than
// the holder, clear it otherwise.
void update_yield(Gate &g) {
    bool ask = false;
    if (g.busy)
        for (const auto &w : g.waiting)
            if (w.second * kYieldRatio < g.holder_weight) {
                ask = true;
                break;
            }
    if (!g.word) return;
    static const bool verbose = std::getenv("BT_PEEL_VERBOSE") != nullptr;
    if (verbose && (g.word[0] != 0) != ask)
        std::fprintf(stderr, "[peel] yield word %d (holder weight %lld, %zu waiting)\n", ask ? 1 : 0,
                     (long long)g.holder_weight, g.waiting.size());
    __atomic_store_n(&g.word[0], ask ? 1 : 0, __ATOMIC_RELEASE);
}

// Under g.mu, with `ticket` in g.waiting: waits for it to be the oldest
// waiter while the device is free, then takes the turn.
void take_turn(Gate &g, std::unique_lock<std::mutex> &lk, uint64_t ticket, int64_t weight) {
    update_yield(g);
    g.cv.wait(lk, [&] { return !g.busy && g.waiting.begin()->first == ticket; });
    g.waiting.erase(ticket);
    g.busy = true;
    g.leaves = false;
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
    g.waiting[ticket_] = weight_;
    if (barriers) {
        take_turn(g, lk, ticket_, weight_);
        return;
    }
    update_yield(g);
    g.cv.wait(lk, [&] {
        return g.busy ? g.leaves : g.waiting.begin()->first == ticket_;
    });
    if (g.busy) {
        held_ = false;
        g.waiting.erase(ticket_);
        update_yield(g);
        g.cv.notify_all();  // the oldest waiter may be another now
    } else {
        take_turn(g, lk, ticket_, weight_);
        g.leaves = true;
        g.cv.notify_all();
    }
}

void CoopTurn::leaves_only() {
    Gate &g = gate();
    std::lock_guard<std::mutex> lk(g.mu);
    g.leaves = true;
    g.cv.notify_all();
}

CoopTurn::~CoopTurn() {
    if (!held_) return;
    Gate &g = gate();
    std::lock_guard<std::mutex> lk(g.mu);
    g.busy = false;
    g.holder_weight = 0;
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
    take_turn(g, lk, ticket_, weight_);
}

}  // namespace bt
