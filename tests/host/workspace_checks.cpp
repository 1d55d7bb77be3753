// workspace_checks.cpp -- checks of the threads' kept memory (csrc/workspace.cpp)
// against a test double of the HIP calls it makes; built with g++ and run by
// tests/test_workspace.py.
//
//   workspace_checks capture  -- no release outside the relaxed capture mode:
//                                it would end another thread's capture
//   workspace_checks devices  -- a thread that goes from device to device keeps
//                                its memory on each
//   workspace_checks waits    -- no call that waits for all of a device's work,
//                                in growth or at a thread's end, and bounds
//   workspace_checks fork     -- a forked child that exits calls no HIP function
#include <sys/wait.h>
#include <unistd.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

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
bool forked = false;    // a child after fork: no call may come
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

hipError_t give(void *p, bool host, bool async, int on = -1)
{
    if (forked) _exit(3);
    std::lock_guard<std::mutex> lk(mu);
    auto it = live.find(p);
    CHECK(it != live.end());
    if (it == live.end()) return hipErrorOutOfMemory;
    CHECK(it->second.host == host && it->second.async == async);
    CHECK(on < 0 || on == it->second.dev);
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
    if (fake::forked) _exit(3);
    std::swap(*m, fake::mode);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t b) { return fake::take(p, b, false, false); }
hipError_t hipFree(void *p) { return fake::give(p, false, false); }
hipError_t hipMallocAsync(void **p, size_t b, hipStream_t) { return fake::take(p, b, false, true); }
hipError_t hipFreeAsync(void *p, hipStream_t s)
{
    return fake::give(p, false, true, s ? s->dev : -1);
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
    qrt::workspace(dev).reserve(need, host_need, nullptr);
}

static int run_capture()
{
    // growth, the way that follows a failed synchronisation, and the thread's end
    std::thread([] {
        reserve(0, 1 << 20, 1 << 16);
        reserve(0, 8 << 20, 1 << 18);
        CHECK(fake::refused == 0);
        qrt::workspace(0).drop(nullptr);
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

static int run_waits()
{
    const size_t MB = 1 << 20;
    // growth in steps, and the thread's end, with and without its own stream
    for (int own = 0; own < 2; own++)
        std::thread([own] {
            if (own) (void)hipStreamCreateWithFlags(&qrt::workspace(0).stream, hipStreamNonBlocking);
            size_t host_before = 0;
            for (size_t mb = 1; mb <= 64; mb *= 2) {
                reserve(0, mb * MB, mb << 16);
                qrt::Workspace &w = qrt::workspace(0);
                CHECK(w.mem && w.mem_bytes >= mb * MB && w.host_bytes >= mb << 16);
                CHECK(w.host_bytes >= host_before);
                host_before = w.host_bytes;
                CHECK(fake::bytes(false) == w.mem_bytes);
            }
            // more than is kept: what is there stays
            reserve(0, qrt::kKeepBytes + 1, qrt::kKeepHostBytes + 1);
            CHECK(qrt::workspace(0).mem_bytes == 64 * MB && qrt::workspace(0).host_bytes == 4 * MB);
        }).join();
    CHECK(fake::waits == 0);
    CHECK(fake::bytes(false) == 0);
    // the second thread took the first one's host blocks
    CHECK(fake::bytes(true) < 8 * MB);
    // many threads at once that end: device memory is given back, and host
    // blocks up to the bound
    std::atomic<int> have{0};
    std::vector<std::thread> th;
    for (int k = 0; k < 12; k++)
        th.emplace_back([&] {
            reserve(0, MB, 4 * MB);
            have++;
            while (have < 12) std::this_thread::yield();
        });
    for (std::thread &t : th) t.join();
    CHECK(fake::bytes(false) == 0);
    CHECK(fake::bytes(true) <= qrt::kSpareHostBytes);
    // a block of one device is not given to a thread on another
    std::thread([] {
        reserve(1, 1 << 20, 1 << 16);
        CHECK(fake::live[qrt::workspace(1).host].dev == 1);
        // after a wait that failed no other thread gets the block
        unsigned char *const host = qrt::workspace(1).host;
        qrt::workspace(1).drop(nullptr);
        CHECK(!qrt::workspace(1).host && !qrt::workspace(1).mem && !fake::live.count(host));
    }).join();
    return 0;
}

static int run_fork()
{
    reserve(0, 1 << 20, 1 << 16);
    std::fflush(nullptr);
    const pid_t child = fork();
    if (child == 0) {
        fake::forked = true;
        std::exit(0);   // runs the destructors of this thread's objects
    }
    int status = -1;
    CHECK(waitpid(child, &status, 0) == child);
    CHECK(WIFEXITED(status) && WEXITSTATUS(status) == 0);
    return 0;
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "capture") run_capture();
    else if (what == "devices") run_devices();
    else if (what == "waits") run_waits();
    else if (what == "fork") run_fork();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), g_fail ? "FAILED" : "ok");
    return g_fail ? 1 : 0;
}
