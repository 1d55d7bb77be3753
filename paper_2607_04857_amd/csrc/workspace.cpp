// workspace.cpp -- memory that a thread keeps between its lone solves.
#include "workspace.h"

#include <map>

namespace qrt {

namespace {

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// While it lives, the thread may allocate and free although another stream
// captures: in any other mode the call fails and ends that capture, another
// thread's too where it is in the global mode (torch.cuda.graph's default).
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture()
    {
        if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

}  // namespace

void Workspace::release_mem()
{
    if (mem) (void)hipFree(mem);
    mem = nullptr;
    mem_bytes = 0;
}

void Workspace::release_host()
{
    if (host) (void)hipHostFree(host);
    host = host_dev = nullptr;
    host_bytes = 0;
}

void Workspace::release()
{
    if (!mem && !host) return;
    RelaxedCapture relaxed;
    release_mem();
    release_host();
}

void Workspace::reserve(size_t need, size_t host_need)
{
    if (need <= mem_bytes && host_need <= host_bytes) return;
    RelaxedCapture relaxed;
    if (need > mem_bytes && need <= kKeepBytes) {
        release_mem();
        const size_t b = align_up(need, size_t(1) << 20);
        void *p = nullptr;
        if (hipMalloc(&p, b) == hipSuccess) {
            mem = static_cast<unsigned char *>(p);
            mem_bytes = b;
        } else {
            (void)hipGetLastError();
        }
    }
    if (host_need > host_bytes && host_need <= kKeepHostBytes) {
        release_host();
        const size_t b = align_up(host_need, size_t(64) << 10);
        void *p = nullptr, *d = nullptr;
        if (hipHostMalloc(&p, b, hipHostMallocMapped) == hipSuccess) {
            if (hipHostGetDevicePointer(&d, p, 0) == hipSuccess) {
                host = static_cast<unsigned char *>(p);
                host_dev = static_cast<unsigned char *>(d);
                host_bytes = b;
            } else {
                (void)hipHostFree(p);
            }
        }
        if (!host) (void)hipGetLastError();
    }
}

Workspace &workspace(int device)
{
    thread_local std::map<int, Workspace> of_device;
    return of_device[device];
}

}  // namespace qrt
