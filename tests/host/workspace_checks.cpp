// workspace_checks.cpp -- checks of the threads' kept memory (csrc/workspace.cpp)
// against a test double of the HIP calls it makes; built with g++ and run by
// tests/test_workspace.py.
//
//   workspace_checks capture  -- no release outside the relaxed capture mode:
//                                it would end another thread's capture
//   workspace_checks devices  -- a thread that goes from device to device keeps
//                                its memory on each
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>

#include "workspace.h"

static int g_fail = 0;
#define CHECK(cond)                                                                \
    do {                                                                           \
        if (!(cond)) {                                                             \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            if (++g_fail > 20) std::exit(1);                                       \
        }                                                                          \
    } while (0)

// ------------------------------------------------------------- the double
struct FakeStream {
    int dev;
};

namespace fake {

struct Block {
    int dev;
    size_t bytes;
    bool host, async;
};
std::mutex mu;
std::map<void *, Block> live;
int refused = 0;        // calls that a capture in the global mode forbids
int waits = 0;          // releases that wait for all of the device's work
int taken = 0;          // allocations
thread_local int dev = 0;
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

size_t bytes(bool host, int on = -1)
{
    size_t s = 0;
    for (auto &kv : live)
        if (kv.second.host == host && (on < 0 || kv.second.dev == on)) s += kv.second.bytes;
    return s;
}

hipError_t take(void **p, size_t b, bool host, bool async)
{
    std::lock_guard<std::mutex> lk(mu);
    if (mode != hipStreamCaptureModeRelaxed && !async) refused++;
    *p = std::malloc(host ? b : 16);
    live[*p] = {dev, b, host, async};
    taken++;
    return hipSuccess;
}

hipError_t give(void *p, bool host, bool async)
{
    std::lock_guard<std::mutex> lk(mu);
    auto it = live.find(p);
    CHECK(it != live.end());
    if (it == live.end()) return hipErrorOutOfMemory;
    CHECK(it->second.host == host && it->second.async == async);
    if (!async) {
        waits++;
        if (mode != hipStreamCaptureModeRelaxed) refused++;
    }
    live.erase(it);
    std::free(p);
    return hipSuccess;
}

}  // namespace fake

hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *d)
{
    *d = fake::dev;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    fake::dev = d;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    std::swap(*m, fake::mode);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t b) { return fake::take(p, b, false, false); }
hipError_t hipFree(void *p) { return fake::give(p, false, false); }
hipError_t hipMallocAsync(void **p, size_t b, hipStream_t) { return fake::take(p, b, false, true); }
hipError_t hipFreeAsync(void *p, hipStream_t s)
{
    CHECK(!s || s->dev == fake::live[p].dev);
    return fake::give(p, false, true);
}
hipError_t hipHostMalloc(void **p, size_t b, unsigned) { return fake::take(p, b, true, false); }
hipError_t hipHostFree(void *p) { return fake::give(p, true, false); }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned)
{
    *d = p;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = new FakeStream{fake::dev};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

// ------------------------------------------------------------- the checks
static void reserve(int dev, size_t need, size_t host_need)
{
    fake::dev = dev;
    qrt::workspace(dev).reserve(need, host_need);
}

static int run_capture()
{
    // growth, the way that follows a failed synchronisation, and the thread's end
    std::thread([] {
        reserve(0, 1 << 20, 1 << 16);
        reserve(0, 8 << 20, 1 << 18);
        CHECK(fake::refused == 0);
        qrt::workspace(0).release();
        CHECK(fake::refused == 0);
        reserve(0, 1 << 20, 1 << 16);
        CHECK(fake::mode == hipStreamCaptureModeGlobal);
    }).join();
    CHECK(fake::refused == 0);
    // another device
    std::thread([] {
        reserve(0, 1 << 20, 1 << 16);
        reserve(1, 1 << 20, 1 << 16);
        CHECK(fake::mode == hipStreamCaptureModeGlobal);
    }).join();
    CHECK(fake::refused == 0);
    CHECK(fake::bytes(false) == 0);
    return 0;
}

static int run_devices()
{
    std::thread([] {
        reserve(0, 3 << 20, 1 << 16);
        reserve(1, 1 << 20, 1 << 17);
        const int taken = fake::taken;
        for (int k = 0; k < 6; k++) {
            qrt::Workspace &w = qrt::workspace(k % 2);
            unsigned char *const mem = w.mem, *const host = w.host;
            reserve(k % 2, 1 << 20, 1 << 16);
            CHECK(w.mem == mem && w.host == host);
            CHECK(fake::live[w.mem].dev == k % 2);
        }
        CHECK(fake::taken == taken);
        CHECK(fake::bytes(false, 0) == 3 << 20 && fake::bytes(false, 1) == 1 << 20);
    }).join();
    CHECK(fake::bytes(false) == 0);
    return 0;
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "capture") run_capture();
    else if (what == "devices") run_devices();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), g_fail ? "FAILED" : "ok");
    return g_fail ? 1 : 0;
}
