// workspace.h -- memory that a thread keeps between its lone solves.
#pragma once

#include <sys/types.h>
#include <unistd.h>

#include <cstddef>

#include <hip/hip_runtime.h>

namespace qrt {

// Device memory and a mapped host block that a thread keeps, for each device it
// solves on, between its lone solves (an allocation, its release and the
// runtime's trimming at each synchronisation cost more than a small solve: 10
// us, and milliseconds for the 110 MB of a k = 1024 solve's lists).  A call has
// them to itself and is synchronous, so the next one may use another stream.  At
// most kKeepBytes of device memory and kKeepHostBytes of host memory are kept;
// larger jobs allocate their own device memory and copy from pageable memory.
// Given back when the thread ends.
//
// hipFree and hipHostFree wait for everything that runs on the device, other
// threads' streams too, so neither is called within a solve or, as a rule, at a
// thread's end (a call that grew beside 45 ms of another stream's work took all
// of them).  Device memory is stream-ordered.  Host blocks that a thread is done
// with go to the other threads: at most kSpareHostBytes wait in the process.
constexpr size_t kKeepBytes = size_t(128) << 20;
constexpr size_t kKeepHostBytes = size_t(4) << 20;
constexpr size_t kSpareHostBytes = size_t(16) << 20;

struct HostBlock {
    int dev = -1;
    unsigned char *host = nullptr, *host_dev = nullptr;   // host and device address
    size_t bytes = 0;
};

struct Workspace {
    const int dev;
    const pid_t pid = getpid();     // (a forked child gives nothing back)
    hipStream_t stream = nullptr;   // the thread's own on the device (thread_stream)
    unsigned char *mem = nullptr, *host = nullptr, *host_dev = nullptr;
    size_t mem_bytes = 0, host_bytes = 0;

    explicit Workspace(int device) : dev(device) {}
    Workspace(const Workspace &) = delete;
    Workspace &operator=(const Workspace &) = delete;
    // At least `need` bytes of device memory and `host_need` of mapped host
    // memory, for a call on stream s of the device (the current one), which waits
    // for s before it returns; either stays null where it cannot be had (the call
    // then does without it).
    void reserve(size_t need, size_t host_need, hipStream_t s);
    // Give both up after work on s that may not have ended (nothing of them goes
    // to another thread before it has).
    void drop(hipStream_t s);
    ~Workspace();

private:
    void release_mem(hipStream_t s);
    void release_host();
};

// The calling thread's on a device.
Workspace &workspace(int device);

}  // namespace qrt
