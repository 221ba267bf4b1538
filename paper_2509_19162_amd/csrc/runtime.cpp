// Host runtime pieces: HIP error mapping, device buffers, look-back epochs,
// HIP-event kernel profiling.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <iterator>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "../../include/cayleygrowth.h"
#include "internal.h"

namespace cg {

void hip_check(hipError_t e, const char *what, const char *file, int line) {
    if (e == hipSuccess) return;
    char buf[512];
    std::snprintf(buf, sizeof buf, "%s failed: %s (%s:%d)", what, hipGetErrorString(e), file, line);
    throw Error(e == hipErrorOutOfMemory ? CG_E_NOMEM : CG_E_DEVICE, buf);
}

// ---------------------------------------------------------------------------
// Device arena. On this HIP runtime a hipMalloc is fast while little memory is
// held, but a large one takes seconds (245 GB: 1.3 to 6 s), and so do later
// ones once tens of GB are held. So buffers are carved out of regions that
// the library reserves: a first one of 16 GiB (0.3 ms; it holds the bitmask
// engine's S_13 and S_12 with every layer kept), with the first request of 16
// MiB or more, and one of most of the device's memory
// (CG_ARENA_FRACTION of what is free, default 0.85; 0 disables both) once
// something does not fit there. Best fit, split on allocation, coalesced on
// free. A range is
// freed only after its owner's stream has drained, so work still queued on
// the old stream never races with a new owner. Requests the arena cannot
// hold fall back to plain hipMalloc/hipFree.
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kAlign = 1u << 16;
constexpr size_t kArenaMinRequest = 16u << 20;  // smaller buffers also use it once it exists
constexpr size_t kArenaFirst = 16ull << 30;

struct Arena {
    struct Region {
        char *base;
        size_t size;
    };
    std::vector<Region> regions;
    bool tried = false;     // the large region was asked for
    bool external = false;  // the caller's memory (cg_set_workspace): never freed here
    std::map<char *, size_t> by_place;       // free ranges: start -> length
    std::multimap<size_t, char *> by_len;    // free ranges: length -> start
    size_t used = 0;

    bool active() const { return !regions.empty(); }
    size_t reserved() const {
        size_t n = 0;
        for (const Region &r : regions) n += r.size;
        return n;
    }
    bool holds(const char *p) const {
        for (const Region &r : regions)
            if (p >= r.base && p < r.base + r.size) return true;
        return false;
    }
    // (ranges of neighbouring regions stay apart)
    bool starts_region(const char *p) const {
        for (const Region &r : regions)
            if (p == r.base) return true;
        return false;
    }
    void add_region(char *base, size_t size) {
        regions.push_back({base, size});
        insert_free(base, size);
    }
    void insert_free(char *at, size_t len) {
        auto nx = by_place.lower_bound(at);
        if (nx != by_place.end() && at + len == nx->first && !starts_region(nx->first)) {  // merge with the next range
            erase_len(nx->second, nx->first);
            len += nx->second;
            nx = by_place.erase(nx);
        }
        if (nx != by_place.begin()) {
            auto pv = std::prev(nx);
            if (pv->first + pv->second == at && !starts_region(at)) {  // merge with the previous range
                erase_len(pv->second, pv->first);
                at = pv->first;
                len += pv->second;
                by_place.erase(pv);
            }
        }
        by_place[at] = len;
        by_len.emplace(len, at);
    }
    void erase_len(size_t len, char *at) {
        auto r = by_len.equal_range(len);
        for (auto it = r.first; it != r.second; ++it)
            if (it->second == at) {
                by_len.erase(it);
                return;
            }
    }
    char *take(size_t len) {
        auto it = by_len.lower_bound(len);
        if (it == by_len.end()) return nullptr;
        const size_t flen = it->first;
        char *const at = it->second;
        by_len.erase(it);
        by_place.erase(at);
        if (flen > len) insert_free(at + len, flen - len);
        used += len;
        return at;
    }
    // hipFree of every region; none may be in use
    void free_regions() {
        if (!external)
            for (const Region &r : regions) (void)hipFree(r.base);
        *this = Arena{};
    }
};

struct DeviceArenas {
    std::mutex mu;
    std::map<int, Arena> arena;
};

DeviceArenas &arenas() {
    static DeviceArenas *a = new DeviceArenas();  // never destroyed: outlives every user
    return *a;
}

int current_device() {
    int d = 0;
    (void)hipGetDevice(&d);
    return d;
}

double arena_fraction() {
    const char *e = std::getenv("CG_ARENA_FRACTION");
    if (!e) return 0.85;
    const double f = std::atof(e);
    return f < 0 ? 0 : (f > 0.95 ? 0.95 : f);
}

// Returns a pointer inside the device's arena, or nullptr.
void *arena_alloc(int dev, size_t len) {
    std::lock_guard<std::mutex> lk(arenas().mu);
    Arena &A = arenas().arena[dev];
    if (char *p = A.take(len)) return p;
    if (A.tried || (!A.active() && len < kArenaMinRequest)) return nullptr;
    const double frac = arena_fraction();
    size_t free_b = 0, total_b = 0;
    if (frac <= 0 || hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
        A.tried = true;
        return nullptr;
    }
    // of the large region: its share of what is free, the first one included
    const size_t first = A.reserved(), share = (size_t)((double)(free_b + first) * frac);
    size_t want = (share > first ? share - first : 0) / kAlign * kAlign;
    if (!A.active() && len <= kArenaFirst / 4 && want > kArenaFirst)
        want = kArenaFirst;
    else
        A.tried = true;
    void *p = nullptr;
    if (want < len || hipMalloc(&p, want) != hipSuccess) {
        (void)hipGetLastError();
        A.tried = true;
        return nullptr;
    }
    A.add_region((char *)p, want);
    return A.take(len);
}

bool arena_free(int dev, void *p, size_t len) {
    std::lock_guard<std::mutex> lk(arenas().mu);
    auto it = arenas().arena.find(dev);
    if (it == arenas().arena.end() || !it->second.holds((char *)p)) return false;
    it->second.insert_free((char *)p, len);
    it->second.used -= len;
    return true;
}

}  // namespace

void release_cached_device_memory() {
    std::lock_guard<std::mutex> lk(arenas().mu);
    for (auto &kv : arenas().arena) {
        Arena &A = kv.second;
        if (!A.active() || A.used || A.external) continue;  // in use, or the caller's
        A.free_regions();
    }
}

void set_workspace(void *p, size_t bytes) {
    const int dev = current_device();
    std::lock_guard<std::mutex> lk(arenas().mu);
    Arena &A = arenas().arena[dev];
    if (A.used) throw Error(CG_E_BUSY, "device buffers still live in the current workspace");
    A.free_regions();
    if (!p) return;  // back to memory the library reserves itself
    const uintptr_t lo = ((uintptr_t)p + 255) & ~(uintptr_t)255;
    const size_t skip = (size_t)(lo - (uintptr_t)p);
    if (bytes <= skip + kAlign) throw Error(CG_E_INVAL, "workspace smaller than 64 KiB");
    const size_t size = (bytes - skip) / kAlign * kAlign;
    A.external = true;
    A.tried = true;
    A.add_region((char *)lo, size);
}

bool arena_active() {
    const int dev = current_device();
    std::lock_guard<std::mutex> lk(arenas().mu);
    auto it = arenas().arena.find(dev);
    return it != arenas().arena.end() && it->second.active();
}

namespace {
// bytes held by every DevBuf of the process (all devices), and the most
// they held at once since the last reset
std::atomic<uint64_t> g_held{0}, g_peak_held{0};

void count_held(uint64_t add) {
    const uint64_t now = g_held.fetch_add(add) + add;
    uint64_t pk = g_peak_held.load();
    while (now > pk && !g_peak_held.compare_exchange_weak(pk, now)) {
    }
}

// Bytes that the library's buffers may hold together: CG_DEVICE_BYTES (for
// tests of what happens when device memory is short), no limit by default.
uint64_t device_bytes_limit() {
    const char *e = std::getenv("CG_DEVICE_BYTES");
    return e ? std::strtoull(e, nullptr, 10) : ~0ull;
}
size_t under_limit(size_t avail) {
    const uint64_t limit = device_bytes_limit(), held = g_held.load();
    return (size_t)std::min<uint64_t>(avail, limit > held ? limit - held : 0);
}
}  // namespace

size_t device_bytes_available() {
    const int dev = current_device();
    size_t free_b = 0, total_b = 0, largest = 0;
    bool tried = false, active = false;
    {
        std::lock_guard<std::mutex> lk(arenas().mu);
        auto it = arenas().arena.find(dev);
        if (it != arenas().arena.end() && it->second.active()) {
            const Arena &A = it->second;
            largest = A.by_len.empty() ? 0 : A.by_len.rbegin()->first;
            tried = A.tried;
            active = true;
        }
    }
    if (!tried) {
        if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
            (void)hipGetLastError();
            free_b = 0;
        }
        largest = std::max(largest, active ? (size_t)((double)free_b * arena_fraction()) : free_b);
    }
    return under_limit(largest);
}

double plan_factor(const char *name) {
    const char *e = std::getenv(name);
    return e ? std::atof(e) : 1.0;
}

void memory_stats(cg_memory_stats_t *out, bool reset_peak) {
    out->held_bytes = g_held.load();
    out->peak_held_bytes = g_peak_held.load();
    uint64_t reserved = 0;
    {
        std::lock_guard<std::mutex> lk(arenas().mu);
        for (auto &kv : arenas().arena)
            if (!kv.second.external) reserved += kv.second.reserved();
    }
    out->arena_bytes = reserved;
    if (reset_peak) g_peak_held.store(g_held.load());
}

bool DevBuf::ensure(size_t need, double slack) {
    if (need <= bytes && p) return false;
    const size_t old = bytes;
    release();
    size_t want = (size_t)((double)need * slack);
    if (want < need) want = need;
    if (old && want < old + old / 2) want = std::max(need, old + old / 2);  // grow geometrically
    if (arena_active()) want = need;  // re-carving the arena is cheap: no slack
    want = (std::max<size_t>(want, 256) + kAlign - 1) / kAlign * kAlign;
    dev = current_device();
    if (want > under_limit(want)) want = (need + kAlign - 1) / kAlign * kAlign;
    if (want > under_limit(want)) throw Error(CG_E_NOMEM, "beyond CG_DEVICE_BYTES");
    void *q = arena_alloc(dev, want);
    if (q) {
        in_arena = true;
    } else {
        in_arena = false;
        hipError_t e = hipMalloc(&q, want);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            want = (need + kAlign - 1) / kAlign * kAlign;  // retry without slack
            e = hipMalloc(&q, want);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                char buf[160];
                std::snprintf(buf, sizeof buf, "device allocation of %zu bytes failed", want);
                throw Error(CG_E_NOMEM, buf);
            }
        }
    }
    p = q;
    bytes = want;
    count_held(want);
    if (held) held->add(want);
    return true;
}

void DevBuf::release() {
    if (p) {
        if (in_arena) {
            // Work still queued on the owner stream may use the range: wait
            // for it, then hand the range back. (No event is kept for later:
            // the owner stream may be destroyed before anyone would query it.)
            if (hipStreamSynchronize(stream) != hipSuccess) {
                (void)hipGetLastError();
                (void)hipDeviceSynchronize();
            }
            (void)arena_free(dev, p, bytes);
        } else {
            (void)hipFree(p);  // a block of its own; synchronises the device
        }
        g_held.fetch_sub(bytes);
        if (held) held->now -= bytes;
    }
    p = nullptr;
    bytes = 0;
}

namespace {
struct IdleKits {
    std::mutex mu;
    std::vector<HostKit> kits;
};
// never destroyed: the HIP runtime may be gone by then
IdleKits &idle_kits() {
    static IdleKits *k = new IdleKits;
    return *k;
}
void destroy_kit(HostKit &k) {
    if (k.host) (void)hipHostFree(k.host);
    if (k.stream) (void)hipStreamDestroy(k.stream);
    k = HostKit();
}
}  // namespace

HostKit take_kit(size_t bytes, bool with_stream) {
    HostKit k;
    CG_HIP(hipGetDevice(&k.dev));
    {
        IdleKits &idle = idle_kits();
        std::lock_guard<std::mutex> lk(idle.mu);
        size_t best = idle.kits.size();
        for (size_t i = 0; i < idle.kits.size(); ++i) {
            const HostKit &x = idle.kits[i];
            if (x.dev != k.dev || x.bytes < bytes) continue;
            // the smallest that does; with a stream if one is wanted, else without
            auto cost = [&](const HostKit &y) { return 2 * y.bytes + ((y.stream != nullptr) != with_stream ? 1u : 0u); };
            if (best == idle.kits.size() || cost(x) < cost(idle.kits[best])) best = i;
        }
        if (best < idle.kits.size()) {
            k = idle.kits[best];
            idle.kits.erase(idle.kits.begin() + (std::ptrdiff_t)best);
        }
    }
    try {
        if (!k.host) {
            k.bytes = 16384;
            while (k.bytes < bytes) k.bytes *= 2;
            CG_HIP(hipHostMalloc(&k.host, k.bytes, hipHostMallocDefault));
        }
        if (with_stream && !k.stream) CG_HIP(hipStreamCreateWithFlags(&k.stream, hipStreamNonBlocking));
    } catch (...) {
        destroy_kit(k);
        throw;
    }
    return k;
}

void give_kit(HostKit &k, bool idle) {
    if (!k.host && !k.stream) return;
    if (idle && k.bytes <= kMaxKitBytes) {
        IdleKits &all = idle_kits();
        std::lock_guard<std::mutex> lk(all.mu);
        if (all.kits.size() < kMaxIdleKits) {
            all.kits.push_back(k);
            k = HostKit();
            return;
        }
    }
    destroy_kit(k);
}

void release_kits() {
    std::vector<HostKit> gone;
    {
        IdleKits &all = idle_kits();
        std::lock_guard<std::mutex> lk(all.mu);
        gone.swap(all.kits);
    }
    for (HostKit &k : gone) destroy_kit(k);
}

void PipeWork::attach(hipStream_t s) {
    stream = s;
    for (DevBuf *b : buffers()) b->stream = s;
}

void PipeWork::init(hipStream_t s) {
    attach(s);
    hist.ensure(kMaxPasses * 256 * sizeof(uint64_t));
    base.ensure(kMaxPasses * 256 * sizeof(uint64_t));
    small.ensure(32 * sizeof(uint32_t) + 4 * sizeof(uint32_t) + 8 * sizeof(uint64_t) + 256);
    CG_HIP(hipMemsetAsync(small.p, 0, small.bytes, stream));
    CG_HIP(hipMemsetAsync(hist.p, 0, hist.bytes, stream));
}

void PipeWork::ensure_status(uint64_t words) {
    if (status.ensure(words * sizeof(uint64_t), 1.25)) {
        CG_HIP(hipMemsetAsync(status.p, 0, status.bytes, stream));
        epoch = 0;
    }
}

uint32_t PipeWork::next_epoch() {
    if (epoch >= 0xFFFFu) {
        CG_HIP(hipMemsetAsync(status.p, 0, status.bytes, stream));
        epoch = 0;
    }
    return ++epoch;
}

const char *kernel_kind_name(int k) {
    static const char *names[K_NUM] = {"expand",      "digit_hist", "digit_scan", "sort_pass_expand",
                                       "sort_pass",   "dedup_compact", "aux",
                                       "bucket_split", "bucket_dedup", "small_layers",
                                       "bitmap_step"};
    return (k >= 0 && k < K_NUM) ? names[k] : "?";
}

hipEvent_t Profiler::get_event() {
    if (!pool.empty()) {
        hipEvent_t e = pool.back();
        pool.pop_back();
        return e;
    }
    hipEvent_t e;
    CG_HIP(hipEventCreate(&e));
    return e;
}

void Profiler::begin(int kind) {
    if (!on) return;
    Pending p{kind, get_event(), get_event(), 0, 0};
    CG_HIP(hipEventRecord(p.a, stream));
    pending.push_back(p);
}

void Profiler::end(int kind, double alg_bytes, double n_items) {
    if (!on) return;
    Pending &p = pending.back();
    (void)kind;
    p.bytes = alg_bytes;
    p.items = n_items;
    CG_HIP(hipEventRecord(p.b, stream));
}

void Profiler::collect() {
    if (!on) return;
    for (auto &p : pending) {
        float ms = 0;
        CG_HIP(hipEventSynchronize(p.b));
        CG_HIP(hipEventElapsedTime(&ms, p.a, p.b));
        total_ms[p.kind] += ms;
        bytes[p.kind] += p.bytes;
        items[p.kind] += p.items;
        launches[p.kind] += 1;
        pool.push_back(p.a);
        pool.push_back(p.b);
    }
    pending.clear();
}

Profiler::~Profiler() {
    for (auto &p : pending) {
        (void)hipEventDestroy(p.a);
        (void)hipEventDestroy(p.b);
    }
    for (auto e : pool) (void)hipEventDestroy(e);
}

}  // namespace cg
