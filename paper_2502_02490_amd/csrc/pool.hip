// Device memory of the contexts' fields, kept for the next context.  A program that measures on many
// gauge fields creates and destroys a context for each; the driver clears freed memory before it hands
// it out again, so allocating the 1.1 GB of a 24^3 x 48 context afresh every time took 37 ms of the
// 42 ms of a create / destroy pair, against 2 ms with the memory of the previous context.
//
// Nothing is kept until a program has shown that it goes from field to field: the memory of the contexts destroyed
// on a device before another one is created there is freed, as it is where contexts live to the program's end.
// Blocks enter only when no work can touch them any more (the caller has synchronised their device
// or the one stream that used them), so any stream or thread may take them.  The pool holds at most
// 1/32 of the device's memory; a block that kIdle later allocations did not want is freed, and so are
// all of a device's blocks when an allocation on it fails or dirac_release_memory is called.
#include <mutex>
#include <new>
#include <vector>

#include "internal.h"

namespace dl {
namespace {

constexpr long kIdle = 128;  // allocations (a context makes about ten)

struct Block {
    void *p;
    size_t bytes;
    int dev;
    long born;  // value of g_clock when it entered
};
std::mutex g_mu;
std::vector<Block> g_blocks;
long g_clock = 0;
constexpr int kDevices = 64;
bool g_destroyed[kDevices], g_again[kDevices];  // a context was destroyed; another one was created after that

size_t limit(int dev) {  // under g_mu
    static size_t lim[kDevices] = {};
    if (dev < 0 || dev >= kDevices || !g_again[dev]) return 0;
    if (!lim[dev]) {
        size_t free_b = 0, total = 0;
        if (hipMemGetInfo(&free_b, &total) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        lim[dev] = total / 32;
    }
    return lim[dev];
}

}  // namespace

void pool_created() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return;
    std::lock_guard<std::mutex> lk(g_mu);
    g_again[dev] = g_destroyed[dev];
}

void pool_destroyed() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return;
    std::lock_guard<std::mutex> lk(g_mu);
    g_destroyed[dev] = true;
}

void *pool_take(size_t n, size_t *got, int *dev) {
    HIP_CHECK(hipGetDevice(dev));
    std::vector<void *> drop;
    void *p = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        ++g_clock;
        int best = -1;
        for (int k = 0; k < (int)g_blocks.size(); ++k) {
            const Block &b = g_blocks[k];
            if (b.dev == *dev && b.bytes >= n && b.bytes <= n + n / 8 && (best < 0 || b.bytes < g_blocks[best].bytes)) best = k;
        }
        if (best >= 0) {
            p = g_blocks[best].p;
            *got = g_blocks[best].bytes;
            g_blocks.erase(g_blocks.begin() + best);
        }
        for (size_t k = 0; k < g_blocks.size();) {
            if (g_blocks[k].dev == *dev && g_clock - g_blocks[k].born > kIdle) {
                drop.push_back(g_blocks[k].p);
                g_blocks.erase(g_blocks.begin() + k);
            } else {
                ++k;
            }
        }
    }
    for (void *q : drop) (void)hipFree(q);
    if (p) return p;
    *got = n;
    hipError_t e = hipMalloc(&p, n);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        pool_trim(*dev);
        e = hipMalloc(&p, n);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        throw Error(e == hipErrorOutOfMemory ? DIRAC_ENOMEM : DIRAC_EHIP, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    return p;
}

void pool_give(void *p, size_t bytes, int dev) noexcept {
    int cur = -1;
    bool kept = false;
    std::vector<void *> drop;
    if (hipGetDevice(&cur) == hipSuccess && cur == dev) {
        std::lock_guard<std::mutex> lk(g_mu);
        try {
            const size_t lim = limit(dev);
            size_t held = bytes;
            for (const Block &b : g_blocks)
                if (b.dev == dev) held += b.bytes;
            if (bytes <= lim) {
                g_blocks.reserve(g_blocks.size() + 1);
                drop.reserve(g_blocks.size());
                for (size_t k = 0; held > lim;) {  // the oldest go first
                    if (g_blocks[k].dev == dev) {
                        held -= g_blocks[k].bytes;
                        drop.push_back(g_blocks[k].p);
                        g_blocks.erase(g_blocks.begin() + k);
                    } else {
                        ++k;
                    }
                }
                g_blocks.push_back(Block{p, bytes, dev, g_clock});
                kept = true;
            }
        } catch (const std::bad_alloc &) {  // no host memory for the list: the block is freed
        }
    }
    for (void *q : drop) (void)hipFree(q);
    if (!kept) (void)hipFree(p);
}

void pool_trim(int dev) {
    std::vector<void *> drop;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (size_t k = 0; k < g_blocks.size();) {
            if (g_blocks[k].dev == dev) {
                drop.push_back(g_blocks[k].p);
                g_blocks.erase(g_blocks.begin() + k);
            } else {
                ++k;
            }
        }
    }
    for (void *q : drop) (void)hipFree(q);
}

}  // namespace dl
