// Device and pinned host memory kept between calls.
//
// A build or a voxelization takes ten to forty allocations and gives most of
// them back before it returns.  On this driver that costs more than the work:
// a release of 128 MB or more takes 0.25-0.3 ms when it goes well, and after
// some tens of rounds of such calls single allocations and releases stall for
// 50 ms to 2 s.  Measured when blocks were first kept, with nothing else
// changed: a build from 29.6M points 26-48 (by how long the process had run)
// -> 5.5 ms, the voxelization of 117M points 97-140 -> 18.4 ms a call.  So
// released blocks stay in a list per device and later calls take them again.
// What is kept is bounded (POOL_SHARE of the device's memory, POOL_PINNED of
// host memory), and it is given back when the device runs low (looked at when
// something is released), when an allocation of the library finds too little
// memory, when the bound is passed (oldest blocks first) and by
// ba_release_cached_memory.
//
// A block enters the list only after all device work that may use it has
// finished (DevArena::release), so any thread and any stream may take it.
#include <hip/hip_runtime.h>

#include <list>
#include <mutex>
#include <new>
#include <utility>

#include "ba.h"
#include "ba_host.hpp"

namespace ba {

static constexpr int POOL_SHARE = 32;                        // of total device memory: 9 GB of 288 GB
static constexpr int LOW_SHARE = 8;                          // keep nothing while less than this share is free
static constexpr size_t POOL_PINNED = (size_t)128 << 20;
static constexpr size_t POOL_STREAMS = 4;

struct PoolBlock {
    void *p;
    size_t bytes;
    int device;   // -1: pinned host memory
};

struct Pool {
    std::mutex mu;
    std::list<PoolBlock> kept;   // oldest first
    size_t dev_bytes = 0, pinned_bytes = 0;
    std::list<std::pair<hipStream_t, int>> streams;   // (stream, device); creating and destroying one takes 1.3 ms
};

// never destroyed: the runtime may be gone when static destructors run
static Pool &pool() {
    static Pool *p = new Pool();
    return *p;
}

// Block sizes: an eighth of an octave apart, in steps of 16 MB from 128 MB on,
// so that calls of nearly the same size share blocks at little waste.
static size_t rounded(size_t nb) {
    size_t step = 256;
    if (nb > ((size_t)128 << 20)) {
        step = (size_t)16 << 20;
    } else {
        while (step * 16 < nb) step *= 2;
    }
    return (nb + step - 1) / step * step;
}

static hipError_t release_block(const PoolBlock &b) {
    if (b.device < 0) return hipHostFree(b.p);
    (void)hipSetDevice(b.device);
    return hipFree(b.p);
}

// Puts a block on a list, or returns it to the driver where the list cannot
// grow: blocks are released by destructors, which must not throw.
static void list_block(std::list<PoolBlock> &l, const PoolBlock &b) {
    try {
        l.push_back(b);
    } catch (const std::bad_alloc &) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        (void)release_block(b);
        (void)hipSetDevice(dev);
    }
}

// Returns blocks to the driver.  One that it refuses (inside a stream capture
// of this thread) goes back to the list, so that it is not lost.
static void give_back(std::list<PoolBlock> &out) {
    if (out.empty()) return;
    int dev = 0;
    (void)hipGetDevice(&dev);
    for (auto it = out.begin(); it != out.end();) {
        if (release_block(*it) == hipSuccess) {
            it = out.erase(it);
        } else {
            (void)hipGetLastError();
            ++it;
        }
    }
    (void)hipSetDevice(dev);
    if (out.empty()) return;
    Pool &P = pool();
    std::lock_guard<std::mutex> lk(P.mu);
    for (const PoolBlock &b : out) (b.device < 0 ? P.pinned_bytes : P.dev_bytes) += b.bytes;
    P.kept.splice(P.kept.begin(), out);
}

// Takes the smallest kept block of at least nb bytes and at most a quarter
// more (so that a small request does not hold a large block).
static void *take(size_t nb, int device, size_t *bytes) {
    Pool &P = pool();
    std::lock_guard<std::mutex> lk(P.mu);
    auto best = P.kept.end();
    for (auto it = P.kept.begin(); it != P.kept.end(); ++it)
        if (it->device == device && it->bytes >= nb && it->bytes <= nb + nb / 4 &&
            (best == P.kept.end() || it->bytes < best->bytes))
            best = it;
    if (best == P.kept.end()) return nullptr;
    void *p = best->p;
    *bytes = best->bytes;
    (device < 0 ? P.pinned_bytes : P.dev_bytes) -= best->bytes;
    P.kept.erase(best);
    return p;
}

void pool_trim() {
    Pool &P = pool();
    std::list<PoolBlock> out;
    std::list<std::pair<hipStream_t, int>> streams;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        out.swap(P.kept);
        streams.swap(P.streams);
        P.dev_bytes = P.pinned_bytes = 0;
    }
    give_back(out);
    for (auto &s : streams) (void)hipStreamDestroy(s.first);
}

// hipMalloc, and for a lack of memory once more without what is kept.
hipError_t device_alloc(void **p, size_t nb) {
    const hipError_t e = hipMalloc(p, nb);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    pool_trim();
    return hipMalloc(p, nb);
}

hipError_t pool_alloc(void **p, size_t nb, size_t *bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t want = rounded(nb);
    if ((*p = take(want, dev, bytes))) return hipSuccess;
    *bytes = want;
    e = hipMalloc(p, want);
    // Only a lack of memory is a reason to give up what is kept: another error
    // (inside a stream capture this thread may neither allocate nor release)
    // would meet the releases too.
    if (e != hipErrorOutOfMemory) return e;
    // once more without what is kept, and without the rounding
    (void)hipGetLastError();
    pool_trim();
    *bytes = nb;
    return hipMalloc(p, nb);
}

// Every device use of the blocks has finished.
void pool_free(const std::vector<DevBlock> &blocks) {
    if (blocks.empty()) return;
    int dev = 0;
    size_t fr = 0, total = 0;
    const bool known = hipGetDevice(&dev) == hipSuccess && hipMemGetInfo(&fr, &total) == hipSuccess;
    Pool &P = pool();
    std::list<PoolBlock> in, out;
    for (const DevBlock &b : blocks) list_block(in, PoolBlock{b.p, b.bytes, b.device});
    {
        std::lock_guard<std::mutex> lk(P.mu);
        while (!in.empty()) {
            const PoolBlock &k = in.front();
            if (!known || k.device != dev || fr < total / LOW_SHARE || k.bytes > total / POOL_SHARE) {
                out.splice(out.end(), in, in.begin());
                continue;
            }
            P.dev_bytes += k.bytes;
            P.kept.splice(P.kept.end(), in, in.begin());
        }
        const size_t bound = known && fr >= total / LOW_SHARE ? total / POOL_SHARE : 0;
        for (auto it = P.kept.begin(); it != P.kept.end() && P.dev_bytes > bound;) {
            if (it->device < 0) {
                ++it;
                continue;
            }
            P.dev_bytes -= it->bytes;
            out.splice(out.end(), P.kept, it++);
        }
    }
    give_back(out);
}

hipError_t pinned_alloc(void **p, size_t nb, size_t *bytes) {
    const size_t want = rounded(nb);
    if ((*p = take(want, -1, bytes))) return hipSuccess;
    *bytes = want;
    const hipError_t e = hipHostMalloc(p, want, hipHostMallocDefault);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    pool_trim();
    return hipHostMalloc(p, want, hipHostMallocDefault);
}

void pinned_free(void *p, size_t bytes) {
    if (!p) return;
    Pool &P = pool();
    std::list<PoolBlock> out;
    list_block(out, PoolBlock{p, bytes, -1});
    if (out.empty()) return;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        if (P.pinned_bytes + bytes <= POOL_PINNED) {
            P.pinned_bytes += bytes;
            P.kept.splice(P.kept.end(), out);
        }
    }
    give_back(out);
}

hipError_t stream_take(hipStream_t *s, int device) {
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lk(P.mu);
        for (auto it = P.streams.begin(); it != P.streams.end(); ++it)
            if (it->second == device) {
                *s = it->first;
                P.streams.erase(it);
                return hipSuccess;
            }
    }
    return hipStreamCreateWithFlags(s, hipStreamNonBlocking);
}

void stream_put(hipStream_t s, int device) {
    if (!s) return;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lk(P.mu);
        if (P.streams.size() < POOL_STREAMS) {
            try {
                P.streams.emplace_back(s, device);
                return;
            } catch (const std::bad_alloc &) {
            }
        }
    }
    (void)hipStreamDestroy(s);
}

void DevArena::release() {
    if (ptrs.empty()) {
        bytes = 0;
        return;
    }
    if (!drained) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        int synced = -1;
        for (const DevBlock &b : ptrs) {
            if (b.device == synced) continue;
            synced = b.device;
            (void)hipSetDevice(synced);
            (void)hipDeviceSynchronize();
        }
        (void)hipSetDevice(dev);
    }
    pool_free(ptrs);
    ptrs.clear();
    slab = nullptr;
    slab_left = 0;
    bytes = 0;
}

ba_status DevArena::alloc_block(void **p, size_t nb) {
    DevBlock b{nullptr, 0, 0};
    try {
        ptrs.reserve(ptrs.size() + 1);   // no block without a place to note it
    } catch (const std::bad_alloc &) {
        set_error("host allocation failed");
        return BA_E_NOMEM;
    }
    (void)hipGetDevice(&b.device);
    hipError_t e = pool_alloc(&b.p, nb, &b.bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        set_error("device allocation of %zu bytes failed: %s", nb, hipGetErrorString(e));
        return BA_E_NOMEM;
    }
    ptrs.push_back(b);
    bytes += b.bytes;
    *p = b.p;
    return BA_OK;
}

}  // namespace ba

extern "C" ba_status ba_release_cached_memory(void) {
    ba::pool_trim();
    return BA_OK;
}
