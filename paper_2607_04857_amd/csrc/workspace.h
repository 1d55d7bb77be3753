// workspace.h -- memory that a thread keeps between its lone solves.
#pragma once

#include <cstddef>

#include <hip/hip_runtime.h>

namespace qrt {

// Device memory and a mapped host block that a thread keeps, for each device it
// solves on, between its lone solves (an allocation, its release and the runtime's trimming at each
// synchronisation cost more than a small solve: 10 us, and milliseconds for
// the 110 MB of a k = 1024 solve's lists).  A call has them to itself and is
// synchronous, so the next one may use another stream.  At most kKeepBytes of
// device memory and kKeepHostBytes of host memory are kept; larger jobs
// allocate their own device memory and copy from pageable memory.  Given back
// when the thread ends.
constexpr size_t kKeepBytes = size_t(128) << 20;
constexpr size_t kKeepHostBytes = size_t(4) << 20;

struct Workspace {
    unsigned char *mem = nullptr, *host = nullptr, *host_dev = nullptr;
    size_t mem_bytes = 0, host_bytes = 0;

    // At least `need` bytes of device memory (of the current device) and
    // `host_need` of mapped host memory; either stays null where it cannot be
    // had (the call then does without it).
    void reserve(size_t need, size_t host_need);
    void release();
    ~Workspace() { release(); }

private:
    void release_mem();
    void release_host();
};

// The calling thread's on a device.
Workspace &workspace(int device);

}  // namespace qrt
