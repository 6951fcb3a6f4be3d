// Host-only program: the library on two devices that are not there.  It defines the HIP calls that
// the library makes (they come before the runtime's, this being the program), counts what was asked
// of each device, and checks
//   lds     that a kernel launched with more dynamic LDS than the default had its limit raised on the
//           device of the launch, and that what one device was asked for the other is asked for too
//   memory  that blocks kept for later handles are released when an allocation needs their room
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <utility>
#include <vector>

#include "handle.h"
#include "internal.h"
#include "newton.h"
#include "serve.h"

static int fails = 0;
#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
            ++fails;                                                          \
        }                                                                     \
    } while (0)

namespace {

std::mutex mu;
thread_local int device = 0;
thread_local hipError_t last_error = hipSuccess;
thread_local size_t launch_lds = 0;
std::map<std::pair<int, const void *>, size_t> limit;   // dynamic LDS allowed, by device and kernel
std::vector<const void *> over;                         // launched beyond it
int launches = 0;
size_t room[2] = {SIZE_MAX, SIZE_MAX}, pinned_room = SIZE_MAX;
std::map<void *, std::pair<int, size_t>> blocks;        // device (-1: pinned host memory) and bytes

constexpr size_t kDefaultLds = 64 * 1024;

hipError_t result(hipError_t e)
{
    if (e != hipSuccess) last_error = e;
    return e;
}

hipError_t allocate(void **p, size_t bytes, int dev)
{
    std::lock_guard<std::mutex> lock(mu);
    size_t &left = dev < 0 ? pinned_room : room[dev];
    if (bytes > left) return result(hipErrorOutOfMemory);
    left -= bytes;
    *p = std::malloc(16);
    blocks[*p] = {dev, bytes};
    return hipSuccess;
}

hipError_t release(void *p)
{
    std::lock_guard<std::mutex> lock(mu);
    const auto it = blocks.find(p);
    if (it == blocks.end()) return p ? result(hipErrorInvalidValue) : hipSuccess;
    (it->second.first < 0 ? pinned_room : room[it->second.first]) += it->second.second;
    std::free(p);
    blocks.erase(it);
    return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipSetDevice(int d) { device = d; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes) { return allocate(p, bytes, device); }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return allocate(p, bytes, -1); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostFree(void *p) { return release(p); }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *fn, hipFuncAttribute, int v)
{
    std::lock_guard<std::mutex> lock(mu);
    limit[{device, fn}] = (size_t)v;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t) { launch_lds = lds; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = *b = dim3(1);
    *lds = launch_lds;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **, size_t lds, hipStream_t)
{
    std::lock_guard<std::mutex> lock(mu);
    ++launches;
    const auto it = limit.find({device, fn});
    if (lds > (it == limit.end() ? kDefaultLds : it->second)) over.push_back(fn);
    return hipSuccess;
}
}

using namespace coxmi;

static void all_launchers(int dev)
{
    (void)hipSetDevice(dev);
    for (const int p : {100, 150, 300, 4096}) {
        CHECK(chol_solve(nullptr, p, nullptr, nullptr, 0, nullptr, nullptr, nullptr) == 0);
        CHECK(prox_model_solve(nullptr, p, nullptr, nullptr, nullptr, nullptr, 0.0, 1, nullptr, nullptr, nullptr) == 0);
        const double c = 0.0;
        for (const bool blocked : {false, true})
            CHECK(syrk_bf16(nullptr, 64, p, blocked, nullptr, nullptr, 64, 8, nullptr, 1.0, 0, nullptr, nullptr) == 0);
        CHECK(syrk_bf16(nullptr, 64, p, false, nullptr, &c, 64, 8, nullptr, 1.0, 0, nullptr, nullptr) == 0);
        CHECK(syrk_fp8(nullptr, 64, p, nullptr, &c, 64, 8, nullptr, nullptr, nullptr, 1.0, 0, nullptr, nullptr) == 0);
    }
    for (int k = 0; k < 3; ++k) {
        FullEvalArgs A;
        A.ld = 512;
        A.p = 200;
        A.max_blocks = 512;
        A.nseg = 1;
        A.seg_rows = 512;
        A.want_xbar = k > 0;
        A.ztype = k == 2 ? kZBF16 : kZF64;
        CHECK(full_eval_launch(A, nullptr) == 0);
    }
    int grid = 0;
    CHECK(serve::launch_step(nullptr, nullptr, 1, 100, nullptr) == 0);
    CHECK(serve::round_grid(100, &grid) == 0);
}

static void lds()
{
    std::thread a([] { all_launchers(0); });   // two devices from two threads, then the other way round
    a.join();
    std::thread b([] { all_launchers(1); });
    b.join();
    std::set<const void *> asked[2];
    for (const auto &l : limit) asked[l.first.first].insert(l.first.second);
    CHECK(launches > 0 && !asked[0].empty());
    CHECK(asked[0] == asked[1]);
    CHECK(over.empty());
}

static void memory()
{
    const size_t mb = (size_t)1 << 20;
    pool_handle_born();
    for (const bool pinned : {false, true}) {
        size_t &left = pinned ? pinned_room : room[0];
        left = 100 * mb;
        void *a = nullptr, *b = nullptr, *other = nullptr;
        device = 1;
        CHECK(pool_get(&other, 8 * mb, false) == hipSuccess);
        pool_put(other);   // stays: the other device's memory is of no use here
        device = 0;
        CHECK(pool_get(&a, 60 * mb, pinned) == hipSuccess);
        pool_put(a);
        CHECK(left == 40 * mb);                                 // kept
        CHECK(pool_get(&b, 90 * mb, pinned) == hipSuccess);     // needs its room
        CHECK(hipGetLastError() == hipSuccess);
        CHECK(pool_get(&a, 60 * mb, pinned) != hipSuccess);     // does not fit at all
        (void)hipGetLastError();
        pool_put(b);
        device = 1;
        void *again = nullptr;
        CHECK(pool_get(&again, 8 * mb, false) == hipSuccess && again == other);
        pool_put(again);
        device = 0;
        left = SIZE_MAX / 2;
    }
    pool_handle_gone();
    CHECK(blocks.empty());
}

int main(int argc, char **argv)
{
    if (argc > 1 && !std::strcmp(argv[1], "lds")) lds();
    if (argc > 1 && !std::strcmp(argv[1], "memory")) memory();
    std::puts(fails ? "FAILED" : "OK");
    return fails != 0;
}
