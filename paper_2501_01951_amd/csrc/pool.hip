// Device memory for the library's own arrays (graphs, their scratch, the work arrays of a build or a
// reordering), kept for reuse after their release.
//
// Building the matrix of a 10^6-node graph takes about 4 ms of kernels and allocates 13 arrays for
// it.  Allocating and freeing them through the driver costs 2 ms at its best and 45 to 115 ms once
// a process has cycled a few tens of gigabytes that way (a free of more than 128 MB then takes tens
// of milliseconds).  A released block therefore stays here and goes to the next request it fits.
//
//  - Bounded: at most kMaxCached bytes per device stay cached; the oldest blocks go back to the driver
//    first, blocks larger than half the bound at once, and all of them when an allocation of the
//    library fails or when mixgcn_release_memory is called.
//  - A block is released either on the one stream that may still have work on it queued (the next
//    owner's stream waits for an event recorded there), or with work queued on any stream: the arrays of
//    a graph.  Such a block is handed on after a wait for its device that has succeeded since, which
//    only calls that may wait make.  The runtime refuses it while any stream of the process is being
//    captured; the request then goes to the driver.
//  - Thread safe: one mutex.
//
// The host copies of row pointers are pinned and kept in the same way (at most kMaxHostCached): a copy of 8 MB into
// ordinary memory goes through staging buffers of 1 MB, each waited for and copied once more by the host, 690 us
// against 151 into pinned memory, and the pages of new ordinary memory are cleared on the way (a first build of 11.1 M
// nodes, 89 MB, 26.6 ms against 7.7).  Pinning takes 12 to 500 us up to 89 MB and 2 ms for 600, giving back as long, and
// waits for the device: so blocks are kept, and given back outside the lock.  Graphs are freed while streams are being
// captured, which an allocation or a release that the runtime refuses then would end: both go in relaxed mode.
#include <stdlib.h>

#include <list>
#include <mutex>
#include <unordered_map>

#include "internal.h"

namespace mixgcn {
namespace {

constexpr size_t kMaxCached = (size_t)4 << 30;
constexpr int kPoolDevices = 16;
constexpr size_t kMaxHostCached = (size_t)512 << 20;
// Smaller blocks are ordinary memory: one staging buffer, and pinning takes up to 180 us where none is cached.
constexpr size_t kLeastPinned = (size_t)1 << 20;

struct Block {
    void* p = nullptr;
    size_t bytes = 0;
    int device = 0;
    hipEvent_t ev = nullptr;  // recorded at the release, if work on one stream could still be queued then
    bool any_stream = false;  // work could be queued on any, and the device has not been waited for since
};

struct Pool {
    std::mutex mu;
    std::list<Block> cached;  // oldest first
    std::unordered_map<void*, Block> in_use;
    std::vector<hipEvent_t> events[kPoolDevices];  // spare events of each device
    std::list<Block> host_cached;                  // oldest first
    std::unordered_map<void*, Block> host_in_use;  // pinned ones
};
Pool& pool()
{
    static Pool* p = new Pool;  // never destroyed: graphs may be freed while the process exits
    return *p;
}

// Multiples of between 1/16 and 1/8 of the size, so that slightly different requests share blocks.
size_t round_size(size_t bytes)
{
    size_t step = 512;
    while (step * 16 <= bytes) step *= 2;
    return bytes < step ? step : (bytes + step - 1) / step * step;
}

void to_driver(Pool& P, Block& b)
{
    if (b.ev) {
        (void)hipEventSynchronize(b.ev);
        P.events[b.device].push_back(b.ev);
    }
    (void)hipFree(b.p);
}

// Gives cached blocks of a device back, oldest first, until at most `keep` bytes are left.
void trim(Pool& P, int device, size_t keep)
{
    size_t have = 0;
    for (const Block& b : P.cached)
        if (b.device == device) have += b.bytes;
    for (auto it = P.cached.begin(); it != P.cached.end() && have > keep;) {
        if (it->device != device) {
            ++it;
            continue;
        }
        have -= it->bytes;
        to_driver(P, *it);
        it = P.cached.erase(it);
    }
}

// Memory from the driver; the cache of the device goes back to it where that fails.
hipError_t malloc_or_trim(Pool& P, int device, void** out, size_t bytes)
{
    hipError_t e = hipMalloc(out, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    trim(P, device, 0);
    e = hipMalloc(out, bytes);
    if (e == hipErrorOutOfMemory) (void)hipGetLastError();
    return e;
}

// What a request may do before it takes a block with work queued on it.
enum class Wait {
    kNone,    // nothing: its stream may be being recorded
    kStream,  // make its stream wait
    kHost,    // and wait for the device
};

int take(void** out, size_t bytes, int device, Wait wait, hipStream_t s)
{
    *out = nullptr;
    Pool& P = pool();
    const size_t want = round_size(bytes);
    std::lock_guard<std::mutex> lock(P.mu);
    // the smallest block that fits and is not more than a quarter larger; the newest of equals
    auto best = P.cached.end();
    for (;;) {
        bool waiting = false;
        for (auto it = P.cached.begin(); it != P.cached.end(); ++it) {
            if (it->device != device || it->bytes < want || it->bytes > want + want / 4) continue;
            if (it->any_stream) waiting = true;
            else if ((!it->ev || wait != Wait::kNone) && (best == P.cached.end() || it->bytes <= best->bytes)) best = it;
        }
        if (best != P.cached.end() || !waiting || wait != Wait::kHost) break;
        if (hipDeviceSynchronize() != hipSuccess) {
            (void)hipGetLastError();
            break;
        }
        for (Block& b : P.cached)
            if (b.device == device) b.any_stream = false;
    }
    Block b;
    if (best != P.cached.end()) {
        if (best->ev) {
            MIXGCN_HIP_TRY(hipStreamWaitEvent(s, best->ev, 0));
            P.events[device].push_back(best->ev);
            best->ev = nullptr;
        }
        b = *best;
        P.cached.erase(best);
    } else {
        b.bytes = want;
        b.device = device;
        MIXGCN_HIP_TRY(malloc_or_trim(P, device, &b.p, want));
    }
    P.in_use[b.p] = b;
    *out = b.p;
    return MIXGCN_OK;
}

// What the runtime refuses while a stream is being captured it allows this thread meanwhile.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture()
    {
        if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// Gives pinned blocks back, not under the lock; what cannot be now stays cached.
void host_to_driver(Pool& P, std::list<Block>& blocks)
{
    if (blocks.empty()) return;
    RelaxedCapture relaxed;
    for (auto it = blocks.begin(); it != blocks.end();) {
        if (hipHostFree(it->p) == hipSuccess) {
            it = blocks.erase(it);
        } else {
            (void)hipGetLastError();
            ++it;
        }
    }
    std::lock_guard<std::mutex> lock(P.mu);
    P.host_cached.splice(P.host_cached.begin(), blocks);
}

int device_of_caller(int* dev)
{
    MIXGCN_HIP_TRY(hipGetDevice(dev));
    if (*dev < 0 || *dev >= kPoolDevices) return fail(MIXGCN_EINVAL, "memory pool: device index");
    return MIXGCN_OK;
}

// stream: work on the block may be queued on s only; otherwise on any stream of its device.
void put_back(void* p, bool stream, hipStream_t s)
{
    if (!p) return;
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    const auto it = P.in_use.find(p);
    if (it == P.in_use.end()) return;
    Block b = it->second;
    P.in_use.erase(it);
    b.any_stream = !stream;
    if (stream) {
        std::vector<hipEvent_t>& spare = P.events[b.device];
        if (!spare.empty()) {
            b.ev = spare.back();
            spare.pop_back();
        } else if (hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) {
            b.ev = nullptr;
        }
        if (!b.ev || hipEventRecord(b.ev, s) != hipSuccess) {
            // nothing to order a reuse by
            (void)hipGetLastError();
            if (b.ev) (void)hipEventDestroy(b.ev);
            b.ev = nullptr;
            b.any_stream = true;
        }
    }
    if (b.bytes > kMaxCached / 2) {
        to_driver(P, b);
        return;
    }
    P.cached.push_back(b);
    trim(P, b.device, kMaxCached);
}

}  // namespace

int pool_alloc(void** p, size_t bytes, hipStream_t s)
{
    int dev = 0;
    MIXGCN_TRY(device_of_caller(&dev));
    return take(p, bytes, dev, Wait::kHost, s);
}

int pool_alloc_async(void** p, size_t bytes, hipStream_t s)
{
    int dev = 0;
    MIXGCN_TRY(device_of_caller(&dev));
    // a stream that is being captured cannot wait for events from outside (nor can the status of the null
    // stream be had while another one is)
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool free_stream = hipStreamIsCapturing(s, &status) == hipSuccess && status == hipStreamCaptureStatusNone;
    if (!free_stream) (void)hipGetLastError();
    return take(p, bytes, dev, free_stream ? Wait::kStream : Wait::kNone, s);
}

int pool_alloc_unordered(void** p, size_t bytes)
{
    int dev = 0;
    MIXGCN_TRY(device_of_caller(&dev));
    return take(p, bytes, dev, Wait::kNone, nullptr);
}

int pool_malloc(void** p, size_t bytes)
{
    int dev = 0;
    MIXGCN_TRY(device_of_caller(&dev));
    std::lock_guard<std::mutex> lock(pool().mu);
    MIXGCN_HIP_TRY(malloc_or_trim(pool(), dev, p, bytes));
    return MIXGCN_OK;
}

void pool_free(void* p) { put_back(p, false, nullptr); }
void pool_free_on(void* p, hipStream_t s) { put_back(p, true, s); }

int host_alloc(void** p, size_t bytes)
{
    *p = nullptr;
    Pool& P = pool();
    Block b;
    b.bytes = round_size(bytes);
    {
        std::lock_guard<std::mutex> lock(P.mu);
        auto best = P.host_cached.end();
        for (auto it = P.host_cached.begin(); it != P.host_cached.end(); ++it)
            if (it->bytes >= b.bytes && it->bytes <= b.bytes + b.bytes / 4 &&
                (best == P.host_cached.end() || it->bytes <= best->bytes))
                best = it;
        if (best != P.host_cached.end()) {
            b = *best;
            P.host_in_use[b.p] = b;
            P.host_cached.erase(best);
            *p = b.p;
            return MIXGCN_OK;
        }
    }
    if (b.bytes >= kLeastPinned) {
        RelaxedCapture relaxed;
        if (hipHostMalloc(&b.p, b.bytes, hipHostMallocPortable) == hipSuccess) {
            std::lock_guard<std::mutex> lock(P.mu);
            P.host_in_use[b.p] = b;
            *p = b.p;
            return MIXGCN_OK;
        }
        (void)hipGetLastError();
    }
    *p = malloc(b.bytes);
    return *p ? MIXGCN_OK : fail(MIXGCN_ENOMEM, "host memory");
}

void host_free(void* p)
{
    if (!p) return;
    Pool& P = pool();
    std::list<Block> victims;
    {
        std::lock_guard<std::mutex> lock(P.mu);
        const auto it = P.host_in_use.find(p);
        if (it == P.host_in_use.end()) {
            free(p);
            return;
        }
        // a block larger than the bound does not push out the others
        std::list<Block>& to = it->second.bytes > kMaxHostCached ? victims : P.host_cached;
        to.push_back(it->second);
        P.host_in_use.erase(it);
        size_t have = 0;
        for (const Block& b : P.host_cached) have += b.bytes;
        while (have > kMaxHostCached) {
            have -= P.host_cached.front().bytes;
            victims.splice(victims.end(), P.host_cached, P.host_cached.begin());
        }
    }
    host_to_driver(P, victims);
}

void pool_release()
{
    Pool& P = pool();
    std::list<Block> host;
    {
        std::lock_guard<std::mutex> lock(P.mu);
        host.swap(P.host_cached);
        for (Block& b : P.cached) to_driver(P, b);
        P.cached.clear();
    }
    host_to_driver(P, host);
}

}  // namespace mixgcn
