// The pool of freed device blocks (alcs_pack.cpp) on a stand-in for the HIP runtime that knows which
// blocks the device may still be reading: a block is never handed out before the device has been waited
// for, waits are not repeated, blocks stay on their device, the bounds hold, everything can be given
// back, and several threads may use it.  Runs without a GPU; prints "pool OK" and returns 0.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "alcs_internal.h"

static std::mutex mu;
static std::map<void *, std::pair<size_t, int>> blocks;  // live allocations: bytes, device
static std::map<int, std::set<void *>> reading;          // per device: what its kernels may still read
static int syncs = 0, mallocs = 0, frees = 0;
static size_t limit = (size_t)1 << 40;
static thread_local int device = 0;

#define CHECK(cond)                                                                     \
    do {                                                                                \
        if (!(cond)) {                                                                  \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                               \
        }                                                                               \
    } while (0)

extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipSetDevice(int d) { device = d; return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 2; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 8; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) {
    std::lock_guard<std::mutex> lock(mu);
    ++syncs;
    reading[device].clear();
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
    std::lock_guard<std::mutex> lock(mu);
    size_t all = n;
    for (auto &b : blocks) all += b.second.first;
    if (all > limit) { *p = nullptr; return hipErrorOutOfMemory; }
    ++mallocs;
    *p = std::malloc(1);
    blocks[*p] = {n, device};
    return hipSuccess;
}
hipError_t hipFree(void *p) {  // waits for the device
    std::lock_guard<std::mutex> lock(mu);
    auto it = blocks.find(p);
    CHECK(it != blocks.end() && it->second.second == device);
    reading[device].clear();
    ++frees;
    blocks.erase(it);
    std::free(p);
    return hipSuccess;
}
}
namespace alcs { int add_channel_records(alcs_packed *, void *) { return ALCS_OK; } }

static void *take(size_t bytes) {
    int rc = -1;
    void *p = alcs::device_alloc(bytes, &rc);
    if (!p) { CHECK(rc == ALCS_E_ALLOC); return nullptr; }
    CHECK(rc == ALCS_OK);
    std::lock_guard<std::mutex> lock(mu);
    CHECK(blocks.count(p) && blocks[p].first >= bytes && blocks[p].second == device);
    CHECK(!reading[device].count(p));  // nobody reads what is handed out
    return p;
}
static void drop(void *p) {  // freed while a kernel reads it
    {
        std::lock_guard<std::mutex> lock(mu);
        reading[blocks[p].second].insert(p);
    }
    alcs::device_free(p);
}
static size_t kept_bytes() {
    size_t all = 0;
    for (auto &b : blocks) all += b.second.first;
    return all;
}

int main() {
    const size_t K = 1 << 20;
    // one wait for all blocks freed before it, none without a new free, a new one after
    void *a = take(3 * K), *b = take(5 * K), *c = take(9 * K);
    drop(a); drop(b);
    CHECK(syncs == 0 && frees == 0);
    CHECK(take(3 * K) == a && syncs == 1);
    CHECK(take(5 * K) == b && syncs == 1);
    drop(a);
    CHECK(take(3 * K) == a && syncs == 2);
    drop(c); drop(b);
    CHECK(take(9 * K) == c && syncs == 3);
    drop(c);                                        // after the wait that covered b
    CHECK(take(5 * K) == b && syncs == 3);
    CHECK(take(9 * K) == c && syncs == 4);
    CHECK(mallocs == 3 && frees == 0);
    // a much smaller request does not take a block, nor does one on another device
    drop(c);
    void *d = take(2 * K);
    CHECK(d != c && mallocs == 4);
    device = 1;
    void *e = take(9 * K);
    CHECK(e != c && mallocs == 5);
    drop(e);
    device = 0;
    CHECK(take(9 * K) == c);
    // everything that nobody uses goes back, on the device it belongs to
    drop(c);
    alcs_release_memory();
    CHECK(frees == 2 && device == 0 && blocks.size() == 3);
    drop(a); drop(b); drop(d);
    alcs_release_memory();
    CHECK(blocks.empty());
    alcs::device_free(nullptr);
    // the bounds: blocks and bytes
    std::vector<void *> many;
    for (int i = 0; i < 300; ++i) many.push_back(take(4096));
    for (void *p : many) drop(p);
    CHECK(blocks.size() == 256);
    many.clear();
    for (int i = 0; i < 8; ++i) many.push_back(take(100 * K));
    for (void *p : many) drop(p);
    CHECK(kept_bytes() <= 512 * K);
    void *big = take(300 * K);
    drop(big);                                      // more than half of the bound: not kept
    CHECK(kept_bytes() <= 512 * K && !blocks.count(big));
    alcs_release_memory();
    CHECK(blocks.empty());
    // out of memory: what is kept goes back first
    limit = 64 * K;
    a = take(30 * K); b = take(30 * K);
    drop(a); drop(b);
    CHECK(take(60 * K) && blocks.size() == 1);
    CHECK(!take(60 * K));
    limit = (size_t)1 << 40;
    // threads
    std::vector<std::thread> ts;
    for (int t = 0; t < 4; ++t)
        ts.emplace_back([t, K]() {
            device = t & 1;
            std::vector<void *> mine;
            unsigned x = 12345u + (unsigned)t;
            for (int i = 0; i < 4000; ++i) {
                x = x * 1664525u + 1013904223u;
                if (mine.size() < 4 && (x >> 16) % 3) mine.push_back(take(K + (x >> 20) % 5 * K / 8));
                else if (!mine.empty()) { drop(mine.back()); mine.pop_back(); }
                if ((x >> 8) % 500 == 0) alcs_release_memory();
            }
            for (void *p : mine) drop(p);
        });
    for (std::thread &t : ts) t.join();
    alcs_release_memory();
    CHECK(blocks.size() == 1);
    std::puts("pool OK");
    return 0;
}
