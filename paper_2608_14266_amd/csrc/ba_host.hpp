// Host-side helpers of libba: error text, status plumbing, device arenas.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "ba.h"

namespace ba {

void set_error(const char *fmt, ...);

#define BA_HIP(call)                                                                                   \
    do {                                                                                               \
        hipError_t _e = (call);                                                                        \
        if (_e != hipSuccess) {                                                                        \
            ::ba::set_error("%s: %s (%s:%d)", #call, hipGetErrorString(_e), __FILE__, __LINE__);       \
            return BA_E_HIP;                                                                           \
        }                                                                                              \
    } while (0)

#define BA_TRY(expr)                                                                                   \
    do {                                                                                               \
        ba_status _s = (expr);                                                                         \
        if (_s != BA_OK) return _s;                                                                    \
    } while (0)

// Optional per-kernel timing with HIP events (ba_profile_enable).
void prof_begin(const char *name, hipStream_t s);
void prof_end(hipStream_t s);
struct ProfScope {
    hipStream_t s;
    ProfScope(const char *name, hipStream_t st) : s(st) { prof_begin(name, st); }
    ~ProfScope() { prof_end(s); }
};

// A slot-owned block of device memory that allocations of the calling thread
// are carved from (bump allocation, 256-byte aligned) while it is installed in
// tl_slot_arena; the owner resets `off` when the work that used it is done.
// Allocations that do not fit fall through to the kept blocks.
struct SlotArena {
    char *base = nullptr;
    size_t cap = 0;
    size_t off = 0;
};
extern thread_local SlotArena *tl_slot_arena;

// Blocks kept between calls (ba_mem.hip).
struct DevBlock {
    void *p;
    size_t bytes;
    int device;
};
hipError_t device_alloc(void **p, size_t nb);   // for hipFree, not for the list
hipError_t pool_alloc(void **p, size_t nb, size_t *bytes);
void pool_free(const std::vector<DevBlock> &blocks);
hipError_t pinned_alloc(void **p, size_t nb, size_t *bytes);
void pinned_free(void *p, size_t bytes);
void pool_trim();
hipError_t stream_take(hipStream_t *s, int device);   // a non-blocking stream of the current device
void stream_put(hipStream_t s, int device);           // idle

// A set of device allocations released together (memory carved from an
// installed slot arena is returned by the arena's owner, not here).  Small
// allocations share slabs.  A released block may be taken by any thread and
// stream at once, so release waits for the device unless the owner has set
// `drained`: every stream that used the arena has been synchronised.
struct DevArena {
    static constexpr size_t SLAB = (size_t)2 << 20, SMALL = SLAB / 8, PAGE = 4096;
    std::vector<DevBlock> ptrs;
    char *slab = nullptr;
    size_t slab_left = 0;
    size_t bytes = 0;       // of the blocks held (a block from the list may be a quarter larger than asked for)
    bool drained = false;
    DevArena() = default;
    DevArena(const DevArena &) = delete;
    DevArena &operator=(const DevArena &) = delete;
    ~DevArena() { release(); }
    void release();
    ba_status alloc_block(void **p, size_t nb);
    size_t used() const { return bytes - slab_left; }   // the blocks without the last slab's free end
    template <class T>
    ba_status alloc(T **p, int64_t count) {
        const size_t nb = sizeof(T) * (size_t)(count > 0 ? count : 1);
        const size_t nba = (nb + 255) / 256 * 256;
        if (SlotArena *a = tl_slot_arena) {
            if (a->off + nba <= a->cap) {
                *p = (T *)(a->base + a->off);
                a->off += nba;
                bytes += nba;
                return BA_OK;
            }
        }
        void *q = nullptr;
        if (nba <= SMALL) {
            const size_t take = (nb + PAGE - 1) / PAGE * PAGE;
            if (take > slab_left) {
                BA_TRY(alloc_block(&q, SLAB));
                slab = (char *)q;
                slab_left = SLAB;
            }
            q = slab;
            slab += take;
            slab_left -= take;
        } else {
            BA_TRY(alloc_block(&q, nb));
        }
        *p = (T *)q;
        return BA_OK;
    }
};

}  // namespace ba
