// Device memory of plans and of the setup calls, kept for the next plan instead of going back to the driver.
//
// Mini-batch training builds two plans for every subgraph and drops them after one step.  hipMalloc and hipFree take
// 10 to 30 us each on this stack, hipFree waits for the device besides, and such a step made about 40 of either: of
// 5.0 ms for a subgraph of 61,226 vertices and 3.1 M edges, 2.5 ms were the GPU waiting for them and for small copies.
//
// A block comes back in one of two ways.  gnn_dev_free_on: its last use is ordered on a stream, an event recorded there
// says when it may be used again (another stream waits for that event on the device, not on the host).  gnn_dev_free:
// any stream may still be using it, as with hipFree; it is handed out again only after a device synchronisation, which
// the next allocation that finds nothing else makes, for all such blocks at once.
//
// What is kept is bounded: GNN_CACHED_MEMORY_BYTES per device, blocks of up to kMaxBlock bytes, and none that has not been asked
// for in kMaxAge allocations.  An allocation that the driver refuses gives everything back first and tries again.
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "common.h"

namespace {

constexpr size_t kMaxIdleBytes = size_t(GNN_CACHED_MEMORY_BYTES);
constexpr size_t kMaxBlock = size_t(GNN_POOL_MAX_BLOCK);
constexpr uint64_t kMaxAge = 4096;
constexpr size_t kHostBlock = GNN_HOST_BLOCK_BYTES;
constexpr size_t kMaxHostBlocks = 16;

struct Block {
    void *p = nullptr;
    size_t bytes = 0;
    hipEvent_t ready = nullptr;  // belongs to the block; meaningful while `event` is set
    bool event = false;          // usable once `ready` has passed
    bool pending = false;        // usable after a device synchronisation
    uint64_t stamp = 0;          // when it was given back
};

struct Device {
    std::multimap<size_t, Block> idle;
    size_t idle_bytes = 0;
    uint64_t clock = 0;
};

struct Pool {
    std::mutex m;
    std::unordered_map<void *, std::pair<int, Block>> live;  // blocks handed out (device, block)
    std::map<int, Device> dev;
    std::vector<void *> host;
};

// Never destroyed: plans may be dropped while the process ends, after static objects are gone.
Pool &pool() {
    static Pool *p = [] {
        Pool *q = new Pool;
        q->host.reserve(kMaxHostBlocks);
        return q;
    }();
    return *p;
}

// Sizes in steps of an eighth of the power of two below: the next subgraph's arrays are a little larger or smaller.
size_t size_class(size_t bytes) {
    if (bytes <= 512) return 512;
    int log2 = 63 - __builtin_clzll(bytes);
    const size_t step = size_t(1) << (log2 - 3);
    return (bytes + step - 1) / step * step;
}

void release(const std::vector<Block> &blocks) {  // without the lock: hipFree waits for the device
    for (const Block &b : blocks) {
        if (b.ready) (void)hipEventDestroy(b.ready);
        (void)hipFree(b.p);
    }
}

std::vector<Block> take_all_idle(Device &d) {
    std::vector<Block> out;
    out.reserve(d.idle.size());
    for (auto &kv : d.idle) out.push_back(kv.second);
    d.idle.clear();
    d.idle_bytes = 0;
    return out;
}

// Puts a block into the idle set and returns what has to go.
std::vector<Block> put_idle(Device &d, Block b) {
    b.stamp = ++d.clock;
    d.idle.emplace(b.bytes, b);
    d.idle_bytes += b.bytes;
    std::vector<Block> out;
    for (auto it = d.idle.begin(); it != d.idle.end();) {
        if (d.clock - it->second.stamp > kMaxAge) {
            out.push_back(it->second);
            d.idle_bytes -= it->first;
            it = d.idle.erase(it);
        } else {
            ++it;
        }
    }
    while (d.idle_bytes > kMaxIdleBytes) {
        auto oldest = d.idle.begin();
        for (auto it = d.idle.begin(); it != d.idle.end(); ++it)
            if (it->second.stamp < oldest->second.stamp) oldest = it;
        out.push_back(oldest->second);
        d.idle_bytes -= oldest->first;
        d.idle.erase(oldest);
    }
    return out;
}

int allocate_from(void **out, size_t bytes, bool has_stream, hipStream_t stream) {
    *out = nullptr;
    // what is built into a fresh block must run now and not when a graph is replayed
    if (has_stream && gnn_capturing(stream)) return GNN_ERR_ALLOC;
    if (bytes > kMaxBlock) {
        if (hipMalloc(out, bytes) == hipSuccess) return GNN_OK;
        (void)hipGetLastError();
        *out = nullptr;
        gnn_pool_release();
        if (hipMalloc(out, bytes) == hipSuccess) return GNN_OK;
        *out = nullptr;
        return GNN_ERR_ALLOC;
    }
    const size_t want = size_class(bytes);
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return GNN_ERR_LAUNCH;
    Pool &P = pool();
    Block b;
    for (bool synced = false;; synced = true) {
        uint64_t seen = 0;
        {
            std::lock_guard<std::mutex> lock(P.m);
            Device &d = P.dev[device];
            auto best = d.idle.end();
            bool any_pending = false;
            for (auto it = d.idle.lower_bound(want); it != d.idle.end() && it->first <= 2 * want; ++it) {
                if (it->second.pending) { any_pending = true; continue; }
                if (it->second.event && hipEventQuery(it->second.ready) != hipSuccess) {
                    (void)hipGetLastError();  // not ready yet
                    if (best == d.idle.end()) best = it;
                    continue;
                }
                it->second.event = false;
                best = it;
                break;
            }
            if (best != d.idle.end()) {
                b = best->second;
                P.live[b.p] = {device, b};
                d.idle_bytes -= best->first;
                d.idle.erase(best);
                break;
            }
            if (!any_pending || synced) break;
            seen = d.clock;
        }
        // outside the lock: another thread may have to launch what this waits for
        if (hipDeviceSynchronize() != hipSuccess) { (void)hipGetLastError(); break; }
        std::lock_guard<std::mutex> lock(P.m);
        for (auto &kv : P.dev[device].idle)
            if (kv.second.pending && kv.second.stamp <= seen) kv.second.pending = false;
    }
    if (b.p) {
        if (b.event) {
            const hipError_t e = has_stream ? hipStreamWaitEvent(stream, b.ready, 0) : hipEventSynchronize(b.ready);
            if (e != hipSuccess) { gnn_dev_free(b.p); return GNN_ERR_LAUNCH; }
        }
        *out = b.p;
        return GNN_OK;
    }
    b.bytes = want;
    if (hipMalloc(&b.p, want) != hipSuccess) {
        (void)hipGetLastError();
        gnn_pool_release();
        if (hipMalloc(&b.p, want) != hipSuccess) return GNN_ERR_ALLOC;
    }
    try {
        std::lock_guard<std::mutex> lock(P.m);
        P.live[b.p] = {device, b};
    } catch (const std::bad_alloc &) {
        (void)hipFree(b.p);
        throw;
    }
    *out = b.p;
    return GNN_OK;
}

// The containers may run out of host memory: no exception leaves the library.
int allocate(void **out, size_t bytes, bool has_stream, hipStream_t stream) {
    try {
        return allocate_from(out, bytes, has_stream, stream);
    } catch (const std::bad_alloc &) {
        return GNN_ERR_ALLOC;
    }
}

}  // namespace

bool gnn_capturing(hipStream_t stream) {
    if (!stream) return false;  // the null stream cannot be captured
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(stream, &s) == hipSuccess && s != hipStreamCaptureStatusNone;
}

void gnn_pool_release() {
    Pool &P = pool();
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return;
    std::vector<Block> blocks;
    try {
        std::lock_guard<std::mutex> lock(P.m);
        blocks = take_all_idle(P.dev[device]);
    } catch (const std::bad_alloc &) {  // they stay
    }
    release(blocks);
}

int gnn_dev_alloc_bytes(void **p, size_t bytes, hipStream_t stream) { return allocate(p, bytes, true, stream); }
int gnn_dev_alloc_bytes(void **p, size_t bytes) { return allocate(p, bytes, false, nullptr); }

static void give_back(void *p, bool has_stream, hipStream_t stream) {
    if (!p) return;
    Pool &P = pool();
    int device = 0;
    Block b;
    {
        std::lock_guard<std::mutex> lock(P.m);
        auto it = P.live.find(p);
        if (it != P.live.end()) {
            device = it->second.first;
            b = it->second.second;
            P.live.erase(it);
        }
    }
    if (!b.p) {  // too large to keep
        (void)hipFree(p);
        return;
    }
    b.event = b.pending = false;
    if (has_stream) {
        if (!b.ready && hipEventCreateWithFlags(&b.ready, hipEventDisableTiming) != hipSuccess) b.ready = nullptr;
        b.event = b.ready && hipEventRecord(b.ready, stream) == hipSuccess;
        if (!b.event) (void)hipGetLastError();
    }
    b.pending = !b.event;
    std::vector<Block> out;
    try {
        std::lock_guard<std::mutex> lock(P.m);
        out = put_idle(P.dev[device], b);
    } catch (const std::bad_alloc &) {  // lost, unless it is among the idle ones already
    }
    release(out);
}

void gnn_dev_free(void *p) { give_back(p, false, nullptr); }
void gnn_dev_free_on(void *p, hipStream_t stream) { give_back(p, true, stream); }

void *gnn_host_block() {
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.m);
        if (!P.host.empty()) {
            void *p = P.host.back();
            P.host.pop_back();
            return p;
        }
    }
    void *p = nullptr;
    return hipHostMalloc(&p, kHostBlock, hipHostMallocPortable) == hipSuccess ? p : nullptr;
}

void gnn_host_block_free(void *p) {
    if (!p) return;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.m);
        if (P.host.size() < kMaxHostBlocks) {
            P.host.push_back(p);  // room for all of them was reserved
            return;
        }
    }
    (void)hipHostFree(p);
}

extern "C" GNN_API void gnn_release_cached_memory(void) { gnn_pool_release(); }
