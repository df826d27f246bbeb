// Device memory of the library: every block an index, a workspace, a build, a
// captured step or a server takes comes from here and goes back here.
//
// Blocks of POOL_MIN bytes and more that are given back are kept for the next
// ones: giving memory back to the driver and taking it again costs up to
// 28 ms per GB once it has to be cleared (a 16 Mbp reference indexed and a
// first batch aligned, over and over: 31 ms a pass with 288 GB of fresh memory
// ahead, 60-150 ms after that).  At most POOL_BYTES a device are held, the
// oldest block goes first, and any allocation that fails, of whatever size,
// gives the device's held blocks back and tries again.

#include <hip/hip_runtime_api.h>

#include <deque>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "bwfm_internal.h"

namespace {

constexpr size_t POOL_BYTES = (size_t)8 << 30;
constexpr size_t POOL_MIN = (size_t)1 << 20;   // smaller blocks are not held
constexpr size_t POOL_STEP = (size_t)2 << 20;  // held blocks' sizes are multiples of this

struct Block {
    void *p = nullptr;
    size_t bytes = 0;
    int dev = -1;
};

struct DevPool {
    std::mutex mu;
    std::unordered_map<void *, Block> live;  // blocks handed out (of POOL_MIN and more)
    std::deque<Block> held;                  // blocks given back, oldest first
    size_t bytes_of(int dev) const {
        size_t n = 0;
        for (const auto &b : held) n += b.dev == dev ? b.bytes : 0;
        return n;
    }
    // take the oldest held block of dev (dev < 0: of any device)
    bool pop(int dev, Block &out) {
        for (auto it = held.begin(); it != held.end(); ++it)
            if (dev < 0 || it->dev == dev) {
                out = *it;
                held.erase(it);
                return true;
            }
        return false;
    }
};
DevPool &pool() {
    static DevPool *p = new DevPool;  // never destroyed: the runtime may be gone at exit
    return *p;
}

// Give the held blocks of dev (< 0: of every device) back to the driver.
bool give_back(int dev) {
    DevPool &P = pool();
    bool any = false;
    for (;;) {
        Block b;
        {
            std::lock_guard<std::mutex> g(P.mu);
            if (!P.pop(dev, b)) return any;
        }
        (void)hipFree(b.p);
        any = true;
    }
}

// hipMalloc, once more without the held blocks when it fails
hipError_t take(void **out, size_t bytes, int dev) {
    hipError_t e = hipMalloc(out, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    if (!give_back(dev)) return e;
    e = hipMalloc(out, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

}  // namespace

int bwfm::dev_malloc(void **out, size_t bytes) {
    *out = nullptr;
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    if (bytes < POOL_MIN) return take(out, bytes, dev);
    DevPool &P = pool();
    const size_t want = (bytes + POOL_STEP - 1) / POOL_STEP * POOL_STEP;
    try {
        // the smallest held block that fits and wastes at most a quarter
        std::lock_guard<std::mutex> g(P.mu);
        size_t best = P.held.size();
        for (size_t i = 0; i < P.held.size(); i++) {
            const auto &b = P.held[i];
            if (b.dev == dev && b.bytes >= want && b.bytes - want <= want / 4 &&
                (best == P.held.size() || b.bytes < P.held[best].bytes))
                best = i;
        }
        if (best < P.held.size()) {
            const Block b = P.held[best];
            P.live[b.p] = b;
            P.held.erase(P.held.begin() + (ptrdiff_t)best);
            *out = b.p;
            return hipSuccess;
        }
    } catch (const std::bad_alloc &) {
        return hipErrorOutOfMemory;
    }
    if (hipError_t e = take(out, want, dev)) {
        *out = nullptr;
        return e;
    }
    try {
        std::lock_guard<std::mutex> g(P.mu);
        P.live[*out] = Block{*out, want, dev};
    } catch (const std::bad_alloc &) {
        // a block that is not listed goes straight back to the driver
    }
    return hipSuccess;
}

// Waits for the device's work, as hipFree does, before the block may be
// handed out again.
void bwfm::dev_free(void *p) {
    if (!p) return;
    DevPool &P = pool();
    Block b;
    {
        std::lock_guard<std::mutex> g(P.mu);
        auto it = P.live.find(p);
        if (it != P.live.end()) {
            b = it->second;
            P.live.erase(it);
        }
    }
    int dev = -1;
    if (!b.p || b.bytes > POOL_BYTES / 2 || hipGetDevice(&dev) != hipSuccess || dev != b.dev ||
        hipDeviceSynchronize() != hipSuccess) {
        (void)hipFree(p);
        return;
    }
    try {
        std::lock_guard<std::mutex> g(P.mu);
        P.held.push_back(b);
    } catch (const std::bad_alloc &) {
        (void)hipFree(p);
        return;
    }
    for (;;) {
        Block old;
        {
            std::lock_guard<std::mutex> g(P.mu);
            if (P.bytes_of(dev) <= POOL_BYTES || !P.pop(dev, old)) return;
        }
        (void)hipFree(old.p);
    }
}

size_t bwfm::dev_cached() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> g(pool().mu);
    return pool().bytes_of(dev);
}

extern "C" int bwfm_release_cached(void) {
    give_back(-1);
    return BWFM_OK;
}
