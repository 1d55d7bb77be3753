// workspace.cpp -- memory that a thread keeps between its lone solves.
#include "workspace.h"

#include <map>
#include <mutex>
#include <vector>

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

// Mapped host blocks that no thread has.  Never destroyed: threads may end
// after the process's static objects.
struct SpareBlocks {
    std::mutex mu;
    std::vector<HostBlock> blocks;
    size_t bytes = 0;
};

SpareBlocks &spare()
{
    static SpareBlocks *s = new SpareBlocks();
    return *s;
}

// A block of at least `need` bytes, the smallest spare one or a new one; its
// host is null where none can be had.
HostBlock take_block(int dev, size_t need)
{
    HostBlock b;
    {
        SpareBlocks &s = spare();
        std::lock_guard<std::mutex> lk(s.mu);
        size_t at = s.blocks.size();
        for (size_t k = 0; k < s.blocks.size(); k++)
            if (s.blocks[k].dev == dev && s.blocks[k].bytes >= need &&
                (at == s.blocks.size() || s.blocks[k].bytes < s.blocks[at].bytes))
                at = k;
        if (at < s.blocks.size()) {
            b = s.blocks[at];
            s.blocks.erase(s.blocks.begin() + long(at));
            s.bytes -= b.bytes;
            return b;
        }
    }
    b.dev = dev;
    // (powers of two: a thread whose jobs grow leaves less behind than it has)
    b.bytes = size_t(64) << 10;
    while (b.bytes < need) b.bytes *= 2;
    void *p = nullptr, *d = nullptr;
    if (hipHostMalloc(&p, b.bytes, hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
    } else if (hipHostGetDevicePointer(&d, p, 0) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipHostFree(p);
    } else {
        b.host = static_cast<unsigned char *>(p);
        b.host_dev = static_cast<unsigned char *>(d);
    }
    return b;
}

void give_block(const HostBlock &b)
{
    {
        SpareBlocks &s = spare();
        std::lock_guard<std::mutex> lk(s.mu);
        if (s.bytes + b.bytes <= kSpareHostBytes) {
            s.blocks.push_back(b);
            s.bytes += b.bytes;
            return;
        }
    }
    (void)hipHostFree(b.host);
}

}  // namespace

void Workspace::release_mem(hipStream_t s)
{
    if (mem) (void)hipFreeAsync(mem, s);
    mem = nullptr;
    mem_bytes = 0;
}

void Workspace::release_host()
{
    if (host) give_block({dev, host, host_dev, host_bytes});
    host = host_dev = nullptr;
    host_bytes = 0;
}

void Workspace::drop(hipStream_t s)
{
    RelaxedCapture relaxed;
    release_mem(s);
    if (host) (void)hipHostFree(host);
    host = host_dev = nullptr;
    host_bytes = 0;
}

void Workspace::reserve(size_t need, size_t host_need, hipStream_t s)
{
    if (need <= mem_bytes && host_need <= host_bytes) return;
    RelaxedCapture relaxed;
    if (need > mem_bytes && need <= kKeepBytes) {
        release_mem(s);
        const size_t b = align_up(need, size_t(1) << 20);
        void *p = nullptr;
        if (hipMallocAsync(&p, b, s) == hipSuccess) {
            mem = static_cast<unsigned char *>(p);
            mem_bytes = b;
        } else {
            (void)hipGetLastError();
        }
    }
    if (host_need > host_bytes && host_need <= kKeepHostBytes) {
        release_host();
        const HostBlock b = take_block(dev, host_need);
        if (b.host) {
            host = b.host;
            host_dev = b.host_dev;
            host_bytes = b.bytes;
        }
    }
}

Workspace::~Workspace()
{
    // (in a child forked since, the runtime and its memory are the parent's)
    if ((!mem && !host) || pid != getpid()) return;
    RelaxedCapture relaxed;
    release_host();
    if (!mem) return;
    // the thread's stream on the device, or one for this
    int cur = dev;
    (void)hipGetDevice(&cur);
    if (cur != dev) (void)hipSetDevice(dev);
    hipStream_t s = stream;
    const bool own = !s && hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess;
    release_mem(s);
    (void)hipStreamSynchronize(s);
    if (own) (void)hipStreamDestroy(s);
    if (cur != dev) (void)hipSetDevice(cur);
}

Workspace &workspace(int device)
{
    thread_local std::map<int, Workspace> of_device;
    return of_device.try_emplace(device, device).first->second;
}

}  // namespace qrt
