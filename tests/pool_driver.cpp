// The pool of kept memory (csrc/ba_mem.hip) on the host, over stand-ins of the
// HIP calls it makes that can be told to fail.  One scenario per run, named by
// the first argument; exit status 0 if it holds.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "ba.h"
#include "ba_host.hpp"

// ---------------------------------------------------------------- stand-ins
static std::map<void *, size_t> g_dev, g_pinned;   // what the "driver" holds
static size_t g_total = (size_t)256 << 30, g_used = 0;
static hipError_t g_malloc_error = hipSuccess, g_free_error = hipSuccess, g_host_error = hipSuccess;
static uintptr_t g_next = (uintptr_t)1 << 40;

// ordinary allocations of the host, refused on request
static bool g_no_new = false;
void *operator new(size_t n) {
    void *p = g_no_new ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static hipError_t take(std::map<void *, size_t> &m, void **p, size_t nb) {
    if (g_used + nb > g_total) return hipErrorOutOfMemory;
    *p = (void *)g_next;
    g_next += nb + 4096;
    m[*p] = nb;
    g_used += nb;
    return hipSuccess;
}
static hipError_t drop(std::map<void *, size_t> &m, void *p) {
    if (!m.count(p)) return hipErrorInvalidValue;
    g_used -= m[p];
    m.erase(p);
    return hipSuccess;
}

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *f = g_total - g_used;
    *t = g_total;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t nb) { return g_malloc_error != hipSuccess ? g_malloc_error : take(g_dev, p, nb); }
hipError_t hipFree(void *p) { return g_free_error != hipSuccess ? g_free_error : drop(g_dev, p); }
hipError_t hipHostMalloc(void **p, size_t nb, unsigned) {
    return g_host_error != hipSuccess ? g_host_error : take(g_pinned, p, nb);
}
hipError_t hipHostFree(void *p) { return g_free_error != hipSuccess ? g_free_error : drop(g_pinned, p); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
}

namespace ba {
void set_error(const char *, ...) {}
thread_local SlotArena *tl_slot_arena = nullptr;
}

// ---------------------------------------------------------------- scenarios
#define CHECK(c)                                                                        \
    do {                                                                                \
        if (!(c)) {                                                                     \
            std::fprintf(stderr, "%s:%d: %s does not hold\n", __FILE__, __LINE__, #c); \
            std::exit(1);                                                               \
        }                                                                               \
    } while (0)

static constexpr size_t MB = (size_t)1 << 20;

// Leaves n kept blocks of 40 MB and returns their bytes.
static size_t keep(int n) {
    ba::DevArena a;
    for (int i = 0; i < n; i++) {
        char *p;
        CHECK(a.alloc(&p, 40 * (int64_t)MB) == BA_OK);
    }
    a.release();
    return g_used;
}

// An allocation refused for another reason than a lack of memory, as inside a
// stream capture, where releases are refused too: what is kept stays kept.
static void refused() {
    const size_t kept = keep(3);
    CHECK(kept >= 120 * MB);
    g_malloc_error = g_free_error = hipErrorStreamCaptureUnsupported;
    ba::DevArena a;
    char *p;
    CHECK(a.alloc(&p, 500 * (int64_t)MB) == BA_E_NOMEM);
    g_malloc_error = g_free_error = hipSuccess;
    CHECK(g_used == kept);
    CHECK(a.alloc(&p, 40 * (int64_t)MB) == BA_OK && g_used == kept);   // from the list
    a.release();
    CHECK(ba_release_cached_memory() == BA_OK && g_used == 0);
}

// Releases refused by the driver, on request and past the bound: the blocks
// stay on the list, serve later calls and go back once releases work.
static void unreleased() {
    const size_t kept = keep(3);
    g_free_error = hipErrorStreamCaptureUnsupported;
    CHECK(ba_release_cached_memory() == BA_OK && g_used == kept);
    ba::DevArena a;
    char *p;
    CHECK(a.alloc(&p, 40 * (int64_t)MB) == BA_OK && g_used == kept);   // from the list
    const size_t big = g_total / 64 + MB;   // two of them pass the bound of 1/32
    for (int i = 0; i < 3; i++) CHECK(a.alloc(&p, (int64_t)big) == BA_OK);
    a.release();
    size_t bytes = 0;
    void *q = nullptr;
    CHECK(ba::pinned_alloc(&q, 200 * MB, &bytes) == hipSuccess);   // above the bound of pinned memory
    ba::pinned_free(q, bytes);
    g_free_error = hipSuccess;
    CHECK(ba_release_cached_memory() == BA_OK && g_used == 0);
}

// A lack of memory while blocks are kept: every allocation of the library is
// tried again without them.
static void lack() {
    const size_t room = g_total;
    void *q = nullptr;
    size_t bytes = 0;
    g_total = keep(3) + MB;
    CHECK(ba::device_alloc(&q, 100 * MB) == hipSuccess && g_used == 100 * MB);
    CHECK(hipFree(q) == hipSuccess);
    g_total = room;
    g_total = keep(3) + MB;
    CHECK(ba::pinned_alloc(&q, 100 * MB, &bytes) == hipSuccess && g_used == bytes);
    ba::pinned_free(q, bytes);
    CHECK(ba_release_cached_memory() == BA_OK && g_used == 0);
    g_total = room;
    g_total = keep(3) + MB;
    ba::DevArena a;
    char *p;
    CHECK(a.alloc(&p, 100 * (int64_t)MB) == BA_OK && g_used == 100 * MB);
    CHECK(a.alloc(&p, 100 * (int64_t)MB) == BA_E_NOMEM);
}

// No host memory left while blocks are released (by destructors, as a rule):
// they go back to the driver, and nothing throws.
static void no_host_memory() {
    size_t bytes = 0;
    void *q = nullptr;
    {
        ba::DevArena a;
        char *p;
        for (int i = 0; i < 3; i++) CHECK(a.alloc(&p, 40 * (int64_t)MB) == BA_OK);
        CHECK(ba::pinned_alloc(&q, MB, &bytes) == hipSuccess);
        g_no_new = true;
        ba::pinned_free(q, bytes);
    }
    g_no_new = false;
    CHECK(g_dev.empty() && g_pinned.empty() && g_used == 0);
    ba::DevArena a;
    char *p;
    g_no_new = true;
    const ba_status st = a.alloc(&p, 40 * (int64_t)MB);
    g_no_new = false;
    CHECK(st == BA_E_NOMEM && g_used == 0);
}

// An arena counts the blocks it holds, not the bytes it asked for.
static void held() {
    keep(1);
    ba::DevArena a;
    char *p;
    CHECK(a.alloc(&p, 33 * (int64_t)MB) == BA_OK);   // the kept block of 40 MB
    CHECK(a.used() == 40 * MB && g_used == 40 * MB);
    for (int i = 1; i <= 600; i++) {   // small ones share slabs, by pages
        CHECK(a.alloc(&p, 5000) == BA_OK);
        CHECK(a.used() >= 40 * MB + (size_t)i * 8192 && a.used() <= g_used);
    }
    CHECK(g_used - a.used() < 2 * MB);
    a.release();
    CHECK(a.used() == 0);
}

int main(int argc, char **argv) {
    const std::string s = argc > 1 ? argv[1] : "";
    if (s == "refused") refused();
    else if (s == "unreleased") unreleased();
    else if (s == "lack") lack();
    else if (s == "no_host_memory") no_host_memory();
    else if (s == "held") held();
    else return 2;
    return 0;
}
