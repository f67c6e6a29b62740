// Device workspace of the library's calls: a caching allocator, one per
// device. A released block is kept with the stream it was released on and an
// event recorded there; it is handed out again at once to a request on the
// same stream (stream order makes that safe) and to a request on another
// stream once its event has completed. New blocks come from hipMalloc (sizes
// rounded up to 1 MiB, or 64 MiB above 256 MiB), only when no cached block
// fits, so repeated calls neither map fresh pages nor synchronise the device.
// Cached blocks are held until the process ends or an allocation of the library
// finds no memory; the device holds at most the peak workspace of the calls that
// overlapped.
#include <algorithm>
#include <deque>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "internal.hpp"

namespace pmlsh {
namespace {

constexpr int kMaxDevices = 64;

struct Block {
    size_t size = 0;
    hipStream_t stream = nullptr;   // stream of the last release
    hipEvent_t ready = nullptr;     // recorded on it at the release
};

struct Cache {
    std::mutex mu;
    std::unordered_map<void*, Block> live;      // handed out
    std::multimap<size_t, std::pair<void*, Block>> free_blocks;   // by size
};

Cache g_cache[kMaxDevices];

size_t rounded(size_t bytes) {
    const size_t q = bytes > (size_t(256) << 20) ? size_t(64) << 20 : size_t(1) << 20;
    return (bytes + q - 1) / q * q;
}

Cache& cache_for_current_device() {
    int dev = 0;
    PMLSH_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) fail(PMLSH_EDEVICE, "device ordinal out of range");
    return g_cache[dev];
}

// Frees the cached blocks whose work has ended (c.mu held).
void trim(Cache& c) {
    for (auto it = c.free_blocks.begin(); it != c.free_blocks.end();) {
        Block& b = it->second.second;
        if (hipEventQuery(b.ready) == hipSuccess) {
            (void)hipEventDestroy(b.ready);
            (void)hipFree(it->second.first);
            it = c.free_blocks.erase(it);
        } else {
            ++it;
        }
    }
    (void)hipGetLastError();   // "not ready" of the queries
}

thread_local BuildScratch* t_scratch = nullptr;   // of the build that this thread runs

// Pinned host blocks of one device: handed out, and given back with the event
// after which their last reader is done. Those of at most kPinnedSmall bytes come
// kPinnedSlab to an allocation (one of its own took longer than a call's other
// host work) and are kept, in the order in which they came back; where the
// readers of kPinnedMost of them are still at work, the next one is waited for.
// Larger blocks are allocated on their own; of those that are idle one is kept.
constexpr size_t kPinnedSmall = 65536, kPinnedSlab = 16, kPinnedMost = 64;

struct PinnedBlock {
    void* p = nullptr;
    size_t size = 0;
    hipEvent_t done = nullptr;
};
struct PinnedCache {
    std::mutex mu;
    std::unordered_map<void*, PinnedBlock> live;
    std::vector<PinnedBlock> fresh;         // small, not yet used
    std::deque<PinnedBlock> back, large;
    size_t made = 0;                        // small ones
};
PinnedCache g_pinned[kMaxDevices];

bool idle(const PinnedBlock& b) { return hipEventQuery(b.done) == hipSuccess; }

void event_of(PinnedBlock& b) {
    if (hipEventCreateWithFlags(&b.done, hipEventDisableTiming) != hipSuccess)
        fail(PMLSH_EDEVICE, "hipEventCreate for a pinned block failed");
}

}  // namespace

void* pinned_alloc(size_t bytes) {
    int dev = 0;
    PMLSH_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) fail(PMLSH_EDEVICE, "device ordinal out of range");
    PinnedCache& c = g_pinned[dev];
    PinnedBlock b;
    if (bytes <= kPinnedSmall) {
        bool wait = false;
        {
            std::lock_guard<std::mutex> g(c.mu);
            auto at = c.back.begin();
            if (c.fresh.empty() && (at == c.back.end() || !idle(*at)) && c.made >= kPinnedMost) {
                at = std::find_if(c.back.begin(), c.back.end(), idle);
                wait = at == c.back.end() && !c.back.empty();
                if (wait) at = c.back.begin();
            }
            if (at != c.back.end() && (wait || idle(*at))) {
                b = *at;
                c.back.erase(at);
            } else {
                if (c.fresh.empty()) {
                    char* slab = nullptr;
                    PMLSH_HIP(hipHostMalloc(&slab, kPinnedSlab * kPinnedSmall, hipHostMallocDefault));
                    for (size_t i = 0; i < kPinnedSlab; ++i) {
                        PinnedBlock x;
                        x.p = slab + i * kPinnedSmall;
                        x.size = kPinnedSmall;
                        event_of(x);
                        c.fresh.push_back(x);
                        ++c.made;
                    }
                }
                b = c.fresh.back();
                c.fresh.pop_back();
            }
            (void)hipGetLastError();   // "not ready" of the queries
            c.live[b.p] = b;
        }
        if (wait) PMLSH_HIP(hipEventSynchronize(b.done));
        return b.p;
    }
    std::vector<PinnedBlock> surplus;
    {
        std::lock_guard<std::mutex> g(c.mu);
        bool kept = false;
        for (size_t i = 0; i < c.large.size();) {
            const PinnedBlock x = c.large[i];
            const bool take = !b.p && x.size >= bytes && idle(x);
            if (!take && (!idle(x) || !kept)) {
                kept = kept || idle(x);
                ++i;
                continue;
            }
            c.large.erase(c.large.begin() + (std::ptrdiff_t)i);
            if (take) b = x;
            else surplus.push_back(x);
        }
        (void)hipGetLastError();
        if (b.p) c.live[b.p] = b;
    }
    for (PinnedBlock& x : surplus) {
        (void)hipEventDestroy(x.done);
        (void)hipHostFree(x.p);
    }
    if (b.p) return b.p;
    b.size = bytes;
    event_of(b);
    PMLSH_HIP(hipHostMalloc(&b.p, bytes, hipHostMallocDefault));
    std::lock_guard<std::mutex> g(c.mu);
    c.live[b.p] = b;
    return b.p;
}

void pinned_free(void* p, hipStream_t st) {
    if (!p) return;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
    PinnedCache& c = g_pinned[dev];
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.live.find(p);
    if (it == c.live.end()) return;
    const PinnedBlock b = it->second;
    c.live.erase(it);
    // without an event only a wait tells when the readers are done
    if (hipEventRecord(b.done, st) != hipSuccess) (void)hipStreamSynchronize(st);
    (b.size == kPinnedSmall ? c.back : c.large).push_back(b);
}

void* ws_alloc(size_t bytes, hipStream_t st) {
    Cache& c = cache_for_current_device();
    const size_t want = rounded(bytes ? bytes : 1);
    std::lock_guard<std::mutex> g(c.mu);
    // smallest cached block that fits and is free for this stream
    for (auto it = c.free_blocks.lower_bound(want); it != c.free_blocks.end(); ++it) {
        Block& b = it->second.second;
        if (b.stream == st || hipEventQuery(b.ready) == hipSuccess) {
            void* p = it->second.first;
            c.live[p] = b;
            c.free_blocks.erase(it);
            return p;
        }
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, want);
    if (e == hipErrorOutOfMemory && !c.free_blocks.empty()) {
        // give the cached blocks that are idle back and try once more
        trim(c);
        e = hipMalloc(&p, want);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        fail(e == hipErrorOutOfMemory ? PMLSH_ENOMEM : PMLSH_EDEVICE,
             std::string("hipMalloc of the workspace: ") + hipGetErrorString(e));
    }
    Block b;
    b.size = want;
    if (hipEventCreateWithFlags(&b.ready, hipEventDisableTiming) != hipSuccess) {
        (void)hipFree(p);
        fail(PMLSH_EDEVICE, "hipEventCreate for the workspace failed");
    }
    c.live[p] = b;
    return p;
}

void* ws_alloc_least(int64_t bytes, hipStream_t st, const std::function<bool(int64_t*)>& smaller) {
    for (;;) {
        try {
            return ws_alloc((size_t)bytes, st);
        } catch (const Error& e) {
            if (e.code != PMLSH_ENOMEM || !smaller(&bytes)) throw;
        }
    }
}

void ws_free(void* p, hipStream_t st) {
    if (!p) return;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
    Cache& c = g_cache[dev];
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.live.find(p);
    if (it == c.live.end()) return;
    Block b = it->second;
    c.live.erase(it);
    b.stream = st;
    if (hipEventRecord(b.ready, st) != hipSuccess) {
        // no event: wait for the stream so the block is idle when reused
        (void)hipStreamSynchronize(st);
        (void)hipEventRecord(b.ready, nullptr);
    }
    c.free_blocks.emplace(b.size, std::make_pair(p, b));
}

void* device_malloc(size_t bytes) {
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        (void)BuildScratch::give_up();
        {
            Cache& c = cache_for_current_device();
            std::lock_guard<std::mutex> g(c.mu);
            trim(c);
        }
        e = hipMalloc(&p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        fail(e == hipErrorOutOfMemory ? PMLSH_ENOMEM : PMLSH_EDEVICE,
             "hipMalloc of " + std::to_string(bytes) + " bytes: " + hipGetErrorString(e));
    }
    return p;
}

// The build's largest buffers come to 46 bytes per point and its level lists
// to some 20 more; what does not fit is allocated on its own. Beyond 2 GB (22
// million points) the allocations are short beside the build.
BuildScratch::BuildScratch(int64_t n) {
    const size_t want = std::min<size_t>((size_t)n * 96 + (size_t(1) << 20), size_t(2) << 30);
    if (hipMalloc(&base_, want) != hipSuccess) {
        (void)hipGetLastError();
        base_ = nullptr;
    } else {
        free_[0] = want;
    }
    outer_ = t_scratch;
    t_scratch = this;
}

BuildScratch::~BuildScratch() {
    t_scratch = outer_;
    if (base_) (void)hipFree(base_);
}

// The index's own arrays may need the memory: they come when the temporaries are
// done with, as if those had been allocated one by one.
bool BuildScratch::give_up() {
    BuildScratch* s = t_scratch;
    if (!s || !s->base_ || !s->used_.empty()) return false;
    (void)hipFree(s->base_);   // waits for the work on its pieces
    s->base_ = nullptr;
    s->free_.clear();
    return true;
}

void* BuildScratch::take_piece(size_t bytes) {
    BuildScratch* s = t_scratch;
    if (!s) return nullptr;
    bytes = std::max<size_t>((bytes + 255) & ~size_t(255), 256);
    for (auto it = s->free_.begin(); it != s->free_.end(); ++it) {
        if (it->second < bytes) continue;
        const size_t at = it->first, left = it->second - bytes;
        s->free_.erase(it);
        if (left) s->free_[at + bytes] = left;
        s->used_[at] = bytes;
        return static_cast<char*>(s->base_) + at;
    }
    return nullptr;
}

bool BuildScratch::give_back(void* p) {
    BuildScratch* s = t_scratch;
    if (!s || !s->base_ || static_cast<char*>(p) < static_cast<char*>(s->base_)) return false;
    auto u = s->used_.find((size_t)(static_cast<char*>(p) - static_cast<char*>(s->base_)));
    if (u == s->used_.end()) return false;
    auto f = s->free_.emplace(u->first, u->second).first;
    s->used_.erase(u);
    auto next = std::next(f);
    if (next != s->free_.end() && f->first + f->second == next->first) {
        f->second += next->second;
        s->free_.erase(next);
    }
    if (f != s->free_.begin()) {
        auto prev = std::prev(f);
        if (prev->first + prev->second == f->first) {
            prev->second += f->second;
            s->free_.erase(f);
        }
    }
    return true;
}

}  // namespace pmlsh
