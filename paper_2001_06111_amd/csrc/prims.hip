// prims.hip - device-wide scans, stable radix sort, fills, workspace, the
// device-memory allocator hook.

#include <algorithm>
#include <cstring>
#include <mutex>
#include <unordered_map>

#include "common.h"

namespace bt {

// ------------------------------------------------------------ errors

static thread_local std::string g_last_error;

void set_error(const std::string &msg) { g_last_error = msg; }

}  // namespace bt

extern "C" const char *bt_last_error(void) { return bt::g_last_error.c_str(); }

namespace bt {

// --------------------------------------------------------- memory
// Every device buffer of the library comes from device_alloc: hipMalloc, or
// the caller's hook (bt_set_allocator).  Each live block remembers the hook
// that made it, so a block is always returned to its own allocator even if
// the hook changes meanwhile.

namespace {
struct Hook {
    bt_alloc_fn alloc = nullptr;
    bt_free_fn free = nullptr;
    void *ctx = nullptr;
};
struct Block {
    Hook hook;
    size_t bytes;
    hipStream_t stream;  // stream-ordered block (nullptr: device-wide)
};
std::mutex &alloc_mu() {
    static std::mutex *m = new std::mutex();  // never destroyed: outlives static teardown
    return *m;
}
Hook g_hook;
std::unordered_map<void *, Block> &live_blocks() {
    static auto *m = new std::unordered_map<void *, Block>();
    return *m;
}
}  // namespace

void set_allocator(bt_alloc_fn a, bt_free_fn f, void *ctx) {
    if ((a == nullptr) != (f == nullptr))
        throw Error{BT_EINVAL, "bt_set_allocator needs both functions or neither"};
    std::lock_guard<std::mutex> lk(alloc_mu());
    g_hook = Hook{a, f, ctx};
}

void *device_alloc(size_t bytes, hipStream_t stream) {
    void *p = nullptr;
    if (bytes == 0) bytes = 256;
    Hook h;
    {
        std::lock_guard<std::mutex> lk(alloc_mu());
        h = g_hook;
    }
    if (h.alloc) {
        p = h.alloc(bytes, h.ctx);
        if (!p)
            throw Error{BT_ENOMEM, "device allocation of " + std::to_string(bytes) +
                                       " bytes failed (allocator hook returned NULL)"};
    } else {
        hipError_t e = stream ? hipMallocAsync(&p, bytes, stream) : hipMalloc(&p, bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            throw Error{BT_ENOMEM, "device allocation of " + std::to_string(bytes) +
                                       " bytes failed: " + hipGetErrorString(e)};
        }
    }
    std::lock_guard<std::mutex> lk(alloc_mu());
    live_blocks()[p] = Block{h, bytes, stream};
    return p;
}

void device_free(void *p) {
    if (!p) return;
    Block b{};
    {
        std::lock_guard<std::mutex> lk(alloc_mu());
        auto it = live_blocks().find(p);
        if (it != live_blocks().end()) {
            b = it->second;
            live_blocks().erase(it);
        }
    }
    if (b.hook.free) {
        // A hook may hand the block out again at once (a caching allocator),
        // so no kernel of the library may still use it.
        if (b.stream)
            (void)hipStreamSynchronize(b.stream);
        else
            (void)hipDeviceSynchronize();
        b.hook.free(p, b.bytes, b.hook.ctx);
    } else if (b.stream) {
        (void)hipFreeAsync(p, b.stream);
    } else {
        (void)hipFree(p);
    }
}

Workspace::~Workspace() { close(); }

hipStream_t Workspace::side(int k) {
    if (!side_[k]) BT_HIP(hipStreamCreateWithFlags(&side_[k], hipStreamNonBlocking));
    return side_[k];
}

void Workspace::sync_sides() {
    for (hipStream_t t : side_)
        if (t) (void)hipStreamSynchronize(t);
}

void Workspace::close() {
    release();
    if (!stream_) return;
    (void)hipStreamSynchronize(stream_);
    for (int64_t *h : old_host_) (void)hipHostFree(h);
    old_host_.clear();
    if (host_) (void)hipHostFree(host_);
    host_ = nullptr;
    host_cap_ = 0;
    stream_ = nullptr;
}

void Workspace::use_arena(void *base, size_t cap, int64_t *host, int n_host) {
    release();
    arena_ = static_cast<char *>(base);
    arena_cap_ = cap;
    arena_top_ = 0;
    host_ = host;
    host_cap_ = n_host;
}

void *Workspace::get(const char *name, size_t bytes) {
    bytes = (bytes + 255) & ~size_t(255);
    if (arena_) {
        // Bump allocation; a name asked again for more memory gets a new
        // region (the old one is reclaimed only by release()).
        for (auto &b : bufs_)
            if (b.name == name && b.cap >= bytes) return b.ptr;
        if (arena_top_ + bytes > arena_cap_)
            throw Error{BT_ENOMEM, "the call needs more than the " + std::to_string(arena_cap_) +
                                       "-byte static scratch (" + std::string(name) + ")"};
        Buf nb;
        nb.name = name;
        nb.ptr = arena_ + arena_top_;
        nb.cap = bytes;
        arena_top_ += bytes;
        for (auto &b : bufs_)
            if (b.name == name) {
                b = nb;
                return nb.ptr;
            }
        bufs_.push_back(nb);
        return nb.ptr;
    }
    for (auto &b : bufs_) {
        if (b.name == name) {
            if (b.cap < bytes) {
                device_free(b.ptr);
                b.ptr = nullptr;
                b.cap = 0;
                b.ptr = device_alloc(bytes + bytes / 8, stream_);
                b.cap = bytes + bytes / 8;
            }
            return b.ptr;
        }
    }
    Buf nb;
    nb.name = name;
    nb.ptr = device_alloc(bytes, stream_);
    nb.cap = bytes;
    bufs_.push_back(nb);
    return nb.ptr;
}

void Workspace::release() {
    if (arena_) {
        bufs_.clear();
        arena_top_ = 0;
        return;
    }
    for (auto &g : graphs) (void)hipGraphExecDestroy(g.exec);
    graphs.clear();
    for (auto &b : bufs_) device_free(b.ptr);
    bufs_.clear();
    for (hipStream_t &t : side_) {
        if (t) (void)hipStreamDestroy(t);
        t = nullptr;
    }
    if (stream_) return;  // host scratch stays until the destructor
    if (host_) (void)hipHostFree(host_);
    host_ = nullptr;
    host_cap_ = 0;
}

void Workspace::drop(const char *const *prefixes) {
    if (arena_) return;
    const auto named = [&](const Buf &b) {
        for (const char *const *p = prefixes; *p; ++p)
            if (b.name.compare(0, std::strlen(*p), *p) == 0) return true;
        return false;
    };
    for (Buf &b : bufs_)
        if (named(b)) device_free(b.ptr);
    bufs_.erase(std::remove_if(bufs_.begin(), bufs_.end(), named), bufs_.end());
}

size_t Workspace::bytes() const {
    if (arena_) return arena_top_;
    size_t t = 0;
    for (auto &b : bufs_) t += b.cap;
    return t;
}

int64_t *Workspace::host(int n) {
    if (arena_) {
        if (n > host_cap_) throw Error{BT_ENOMEM, "host scratch of the arena too small"};
        return host_;
    }
    if (n > host_cap_) {
        if (host_) {
            if (stream_)
                old_host_.push_back(host_);
            else
                (void)hipHostFree(host_);
        }
        host_ = nullptr;
        host_cap_ = 0;
        const int cap = n > 4096 ? n : 4096;
        BT_HIP(hipHostMalloc((void **)&host_, sizeof(int64_t) * cap, hipHostMallocDefault));
        host_cap_ = cap;
    }
    return host_;
}

int grid_for(int64_t n, int block, int max_blocks) {
    int64_t g = ceil_div(n, block);
    if (g < 1) g = 1;
    if (g > max_blocks) g = max_blocks;
    return (int)g;
}

// ------------------------------------------------------------ fills

template <typename T> __global__ void k_fill(T *p, T v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    k_fill<int32_t><<<grid_for(n, 256, 8192), 256, 0, s>>>(p, v, n);
    BT_CHECK_LAUNCH();
}
void fill_i64(int64_t *p, int64_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    k_fill<int64_t><<<grid_for(n, 256, 8192), 256, 0, s>>>(p, v, n);
    BT_CHECK_LAUNCH();
}
void fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    k_fill<uint32_t><<<grid_for(n, 256, 8192), 256, 0, s>>>(p, v, n);
    BT_CHECK_LAUNCH();
}

// Clearing by a kernel rather than hipMemsetAsync: a caller may capture the
// library's work in a HIP graph, where memset nodes are avoided.
void zero_bytes(void *p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return;
    if (bytes % 4 != 0 || reinterpret_cast<uintptr_t>(p) % 4 != 0)
        throw Error{BT_EDEVICE, "zero_bytes: size or address not a multiple of 4"};
    fill_u32(static_cast<uint32_t *>(p), 0u, (int64_t)(bytes / 4), s);
}

// ------------------------------------------------------------ scan
// Reduce-then-scan: per-tile sums, a recursive scan of those, then a
// per-tile scan seeded with the tile's offset.  Each thread owns
// kScanItems consecutive elements.

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanBlock * kScanItems;

template <typename Tin>
__global__ __launch_bounds__(kScanBlock) void k_scan_reduce(const Tin *in, int64_t n,
                                                            int64_t *bsum) {
    __shared__ int64_t part[kScanBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t s = 0;
    for (int i = threadIdx.x; i < kScanTile; i += kScanBlock) {
        int64_t idx = base + i;
        if (idx < n) s += (int64_t)in[idx];
    }
    s = wave_sum(s);
    if (lane_id() == 0) part[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kScanBlock / kWave; ++w) t += part[w];
        bsum[blockIdx.x] = t;
    }
}

template <typename Tin>
__global__ __launch_bounds__(kScanBlock) void k_scan_tile(const Tin *in, int64_t *out,
                                                          int64_t n, const int64_t *boff) {
    __shared__ int64_t scratch[kScanBlock / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t idx = base + i;
        v[i] = idx < n ? (int64_t)in[idx] : 0;
        sum += v[i];
    }
    int64_t total;
    int64_t run = block_exclusive_sum(sum, scratch, &total);
    run += boff[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t idx = base + i;
        if (idx < n) out[idx] = run;
        run += v[i];
        if (idx == n - 1) out[n] = run;
    }
}

// Up to kScanOne elements: each workgroup sums what precedes its tile by
// itself, one launch instead of three (a launch costs 3 to 4 us, the sums of
// the last workgroup under 3 us).
constexpr int64_t kScanOne = 16 * kScanTile;

// A second row of workgroups scans in1.
template <typename Tin>
__global__ __launch_bounds__(kScanBlock) void k_scan_one(const Tin *in0, int64_t *out0,
                                                         const Tin *in1, int64_t *out1, int64_t n) {
    const Tin *const in = blockIdx.y ? in1 : in0;
    int64_t *const out = blockIdx.y ? out1 : out0;
    __shared__ int64_t scratch[kScanBlock / kWave + 1];
    const int64_t tile = (int64_t)blockIdx.x * kScanTile;
    int64_t before = 0;
#pragma unroll 8
    for (int64_t i = threadIdx.x; i < tile; i += kScanBlock) before += (int64_t)in[i];
    int64_t off;
    (void)block_exclusive_sum(before, scratch, &off);
    const int64_t base = tile + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = base + i < n ? (int64_t)in[base + i] : 0;
        sum += v[i];
    }
    int64_t total;
    int64_t run = block_exclusive_sum(sum, scratch, &total) + off;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
        if (base + i == n - 1) out[n] = run;
    }
}

template <typename Tin>
static void scan_impl(const Tin *in, int64_t *out, int64_t n, Workspace &ws, hipStream_t s,
                      int level) {
    if (n <= 0) {
        fill_i64(out, 0, 1, s);
        return;
    }
    int64_t nb = ceil_div(n, kScanTile);
    if (n <= kScanOne) {
        k_scan_one<Tin><<<(unsigned)nb, kScanBlock, 0, s>>>(in, out, nullptr, nullptr, n);
        BT_CHECK_LAUNCH();
        return;
    }
    char nb_name[32], no_name[32];
    snprintf(nb_name, sizeof nb_name, "scan_bsum%d", level);
    snprintf(no_name, sizeof no_name, "scan_boff%d", level);
    int64_t *bsum = ws.get<int64_t>(nb_name, nb);
    int64_t *boff = ws.get<int64_t>(no_name, nb + 1);
    k_scan_reduce<Tin><<<(unsigned)nb, kScanBlock, 0, s>>>(in, n, bsum);
    BT_CHECK_LAUNCH();
    scan_impl<int64_t>(bsum, boff, nb, ws, s, level + 1);
    k_scan_tile<Tin><<<(unsigned)nb, kScanBlock, 0, s>>>(in, out, n, boff);
    BT_CHECK_LAUNCH();
}

void scan_exclusive_i64(const int64_t *in, int64_t *out, int64_t n, Workspace &ws,
                        hipStream_t s) {
    scan_impl<int64_t>(in, out, n, ws, s, 0);
}

void scan_exclusive_i32_to_i64(const int32_t *in, int64_t *out, int64_t n, Workspace &ws,
                               hipStream_t s) {
    scan_impl<int32_t>(in, out, n, ws, s, 0);
}

void scan_two_i32_to_i64(const int32_t *in0, int64_t *out0, const int32_t *in1, int64_t *out1,
                         int64_t n, Workspace &ws, hipStream_t s) {
    if (n > 0 && n <= kScanOne) {
        k_scan_one<int32_t><<<dim3((unsigned)ceil_div(n, kScanTile), 2), kScanBlock, 0, s>>>(
            in0, out0, in1, out1, n);
        BT_CHECK_LAUNCH();
        return;
    }
    scan_exclusive_i32_to_i64(in0, out0, n, ws, s);
    scan_exclusive_i32_to_i64(in1, out1, n, ws, s);
}

// ------------------------------------------------------- radix sort
// Stable LSD radix sort.  A pass: per-tile digit histograms, one exclusive
// scan over them, a stable scatter.
//
// The scatter's workgroup loads its whole tile at once and each wave owns a
// run of it: the waves' digit counts give every wave its own output
// positions, so ranking the 64 elements of a row (one ballot a digit bit)
// needs no barrier.  With a tile loaded row by row and three barriers a row a
// pass of 10M elements took 86 us in the scatter, and one of 20,000 15 us;
// now one of 5M takes 38 us and one of 10,000 8 us.  Few tiles (kRsDirect)
// are scanned by the scatter itself, each workgroup for its own, which saves a
// pass its scan launches.
//
// Digits: up to 11 bits up to kRsSmall elements, where a pass costs its two
// launches whatever it moves; up to 8 above, where wide digits write short
// runs (5M-edge graph, six or nine passes: 408 and 340 us in the scatter).

template <int ITEMS> constexpr int kRsDigit = ITEMS == 4 ? 11 : 8;
constexpr int kRsBlock = 256;
constexpr int kRsWaves = kRsBlock / kWave;
constexpr int64_t kRsSmall = int64_t(1) << 16;  // up to here: tiles of 1,024, else of 4,096
constexpr int64_t kRsDirect = 64;

template <int ITEMS>
__global__ __launch_bounds__(kRsBlock) void k_rs_hist(const uint64_t *keys, int64_t n, int shift,
                                                      int bins, bool direct, int32_t *hist,
                                                      int64_t nb) {
    extern __shared__ int32_t h[];
    for (int d = threadIdx.x; d < bins; d += kRsBlock) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (ITEMS * kRsBlock);
    uint64_t k[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = base + i * kRsBlock + threadIdx.x;
        k[i] = idx < n ? keys[idx] : 0;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (base + i * kRsBlock + threadIdx.x < n)
            atomicAdd(&h[(int)(k[i] >> shift) & (bins - 1)], 1);
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kRsBlock)
        hist[direct ? (int64_t)blockIdx.x * bins + d : (int64_t)d * nb + blockIdx.x] = h[d];
}

// offs: the scanned histograms (digit by digit), or null for few tiles, whose
// histograms (tile by tile) are summed here.
template <int ITEMS>
__global__ __launch_bounds__(kRsBlock) void k_rs_scatter(const uint64_t *kin, const uint32_t *vin,
                                                         uint64_t *kout, uint32_t *vout, int64_t n,
                                                         int shift, int bits, const int32_t *hist,
                                                         const int64_t *offs, int64_t nb) {
    extern __shared__ uint32_t wc[];  // [wave][digit]: counts, then output positions
    __shared__ uint32_t scr[kRsWaves + 1];
    const int bins = 1 << bits;
    const int w = threadIdx.x / kWave;
    uint32_t *mine = wc + w * bins;
    const int64_t base = (int64_t)blockIdx.x * (ITEMS * kRsBlock) + w * (ITEMS * kWave);
    uint64_t k[ITEMS];
    uint32_t v[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = base + i * kWave + lane_id();
        k[i] = idx < n ? kin[idx] : 0;
        v[i] = idx < n ? vin[idx] : 0;
    }
    for (int d = threadIdx.x; d < kRsWaves * bins; d += kRsBlock) wc[d] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (base + i * kWave + lane_id() < n) atomicAdd(&mine[(int)(k[i] >> shift) & (bins - 1)], 1u);
    __syncthreads();
    uint32_t *first = wc + kRsWaves * bins;  // few tiles: each digit's first position
    uint32_t before[(1 << kRsDigit<ITEMS>) / kRsBlock];
    if (!offs) {
#pragma unroll
        for (int i = 0; i < (1 << kRsDigit<ITEMS>) / kRsBlock; ++i) {
            const int d = i * kRsBlock + (int)threadIdx.x;
            before[i] = 0;
            if (d >= bins) continue;
            uint32_t total = 0;
#pragma unroll 8
            for (int t = 0; t < (int)nb; ++t) {
                const uint32_t c = (uint32_t)hist[t * bins + d];
                before[i] += t < (int)blockIdx.x ? c : 0;
                total += c;
            }
            first[d] = total;
        }
        __syncthreads();
        const int per = (bins + kRsBlock - 1) / kRsBlock;
        const int d0 = (int)threadIdx.x * per, d1 = min(d0 + per, bins);
        uint32_t sum = 0, all;
        for (int d = d0; d < d1; ++d) sum += first[d];
        uint32_t run = block_exclusive_sum<uint32_t>(sum, scr, &all);
        for (int d = d0; d < d1; ++d) {
            const uint32_t c = first[d];
            first[d] = run;
            run += c;
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < (1 << kRsDigit<ITEMS>) / kRsBlock; ++i) {
        const int d = i * kRsBlock + (int)threadIdx.x;
        if (d >= bins) continue;
        uint32_t pos =
            offs ? (uint32_t)offs[(int64_t)d * nb + blockIdx.x] : first[d] + before[i];
        for (int j = 0; j < kRsWaves; ++j) {
            const uint32_t c = wc[j * bins + d];
            wc[j * bins + d] = pos;
            pos += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = base + i * kWave + lane_id() < n;
        const int d = (int)(k[i] >> shift) & (bins - 1);
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t pos = mine[d] + rank;
        if (valid) {
            kout[pos] = k[i];
            vout[pos] = v[i];
        }
        wave_fence();  // all lanes have read the position
        if (valid && rank == 0) mine[d] = pos + (uint32_t)__popcll(peers);
        wave_fence();
    }
}

template <int ITEMS>
static void radix_passes(uint64_t *&ka, uint32_t *&va, uint64_t *&kb, uint32_t *&vb, int64_t n,
                         int begin, int key_bits, Workspace &ws, hipStream_t s) {
    const int64_t nb = ceil_div(n, ITEMS * kRsBlock);
    const int passes = (key_bits + kRsDigit<ITEMS> - 1) / kRsDigit<ITEMS>;
    const int widest = (key_bits + passes - 1) / passes;
    const bool direct = nb <= kRsDirect;
    int32_t *hist = ws.get<int32_t>("rs_hist", nb << widest);
    int64_t *offs = direct ? nullptr : ws.get<int64_t>("rs_offs", (nb << widest) + 1);
    for (int p = 0, done = 0; p < passes; ++p) {
        const int bits = (key_bits - done + passes - p - 1) / (passes - p);
        const int shift = begin + done, bins = 1 << bits;
        k_rs_hist<ITEMS><<<(unsigned)nb, kRsBlock, sizeof(int32_t) * bins, s>>>(
            ka, n, shift, bins, direct, hist, nb);
        BT_CHECK_LAUNCH();
        if (!direct) scan_exclusive_i32_to_i64(hist, offs, nb << bits, ws, s);
        k_rs_scatter<ITEMS><<<(unsigned)nb, kRsBlock, sizeof(int32_t) * (kRsWaves + 1) * bins, s>>>(
            ka, va, kb, vb, n, shift, bits, hist, offs, nb);
        BT_CHECK_LAUNCH();
        std::swap(ka, kb);
        std::swap(va, vb);
        done += bits;
    }
}

void radix_sort_swap(uint64_t *&keys, uint32_t *&vals, uint64_t *&keys2, uint32_t *&vals2,
                     int64_t n, int key_bits, Workspace &ws, hipStream_t s, int begin) {
    if (n <= 1 || key_bits <= 0) return;
    if (n >> 32) throw Error{BT_EOVERFLOW, "too many elements to sort"};
    if (n <= kRsSmall) radix_passes<4>(keys, vals, keys2, vals2, n, begin, key_bits, ws, s);
    else radix_passes<16>(keys, vals, keys2, vals2, n, begin, key_bits, ws, s);
}

void radix_sort_u64_u32(uint64_t *keys, uint32_t *vals, int64_t n, int key_bits, Workspace &ws,
                        hipStream_t s, int begin) {
    if (n <= 1 || key_bits <= 0) return;
    uint64_t *ka = keys, *kb = ws.get<uint64_t>("rs_keys", n);
    uint32_t *va = vals, *vb = ws.get<uint32_t>("rs_vals", n);
    radix_sort_swap(ka, va, kb, vb, n, key_bits, ws, s, begin);
    if (ka != keys) {
        BT_HIP(hipMemcpyAsync(keys, ka, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, s));
        BT_HIP(hipMemcpyAsync(vals, va, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s));
    }
}

}  // namespace bt
