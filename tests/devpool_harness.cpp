// The library's device-memory pool (csrc/devpool.cpp) on two made-up devices
// of 20 GB each: the few runtime calls it makes are defined here.  Prints
// "all checks passed".
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <map>

#include "../paper_1505_07855_amd/csrc/bwfm_internal.h"

namespace {
constexpr size_t GB = (size_t)1 << 30, CAP = 20 * GB;
struct Mem {
    size_t bytes;
    int dev;
};
std::map<void *, Mem> mem;
int cur = 0;
size_t used(int dev) {
    size_t n = 0;
    for (auto &m : mem) n += m.second.dev == dev ? m.second.bytes : 0;
    return n;
}
void check(bool ok, const char *what) {
    if (!ok) {
        std::printf("failed: %s\n", what);
        std::exit(1);
    }
}
void *get(size_t bytes) {
    void *p = nullptr;
    return bwfm::dev_malloc(&p, bytes) == hipSuccess ? p : nullptr;
}
}  // namespace

hipError_t hipMalloc(void **p, size_t bytes) {
    *p = nullptr;
    if (used(cur) + bytes > CAP) return hipErrorOutOfMemory;
    *p = std::malloc(16);
    mem[*p] = Mem{bytes, cur};
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    check(mem.erase(p) == 1, "only live blocks are freed");
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = cur;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

int main() {
    // a block given back serves the next request of its size
    void *a = get(3 * GB);
    bwfm::dev_free(a);
    check(used(0) == 3 * GB && bwfm::dev_cached() == 3 * GB, "a block is held");
    void *b = get(3 * GB - 1000);
    check(b == a && bwfm::dev_cached() == 0, "a held block is reused");
    bwfm::dev_free(b);
    // an allocation that fails, large or small, has the held blocks back
    void *big = get(18 * GB);
    check(big && used(0) == 18 * GB, "a large allocation after the held blocks went back");
    void *c = get(2 * GB);
    bwfm::dev_free(c);
    void *d = get(4096);
    check(d && used(0) == 18 * GB + 4096, "a small allocation after the held blocks went back");
    check(!get(3 * GB), "what does not fit is refused");
    bwfm::dev_free(big);
    bwfm::dev_free(d);
    check(used(0) == 0, "blocks of more than half the bound and small ones are not held");

    // devices are counted apart
    void *e = get(4 * GB), *f = get(4 * GB);
    bwfm::dev_free(e);
    bwfm::dev_free(f);
    cur = 1;
    check(bwfm::dev_cached() == 0, "another device's held blocks are not this one's");
    void *g = get(3 * GB);
    bwfm::dev_free(g);
    check(used(0) == 8 * GB && used(1) == 3 * GB, "the bound is a device's own");
    check(get(18 * GB) && used(0) == 8 * GB && used(1) == 18 * GB, "a failing device has its own blocks back");
    cur = 0;
    check(bwfm::dev_cached() == 8 * GB, "the first device still holds its blocks");
    // the caller may have all of them back
    check(bwfm_release_cached() == BWFM_OK && used(0) == 0 && bwfm::dev_cached() == 0, "released");
    std::printf("all checks passed\n");
    return 0;
}
