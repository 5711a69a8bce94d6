// Device memory of the host side: blocks kept between calls.
#pragma once
#include <mutex>

#include <hip/hip_runtime.h>

namespace ivf {

// Device memory kept for the next call.  The index-time entry points need scratch of a call's size for a call's time and
// wait for their stream before they return; hipMalloc and hipFree cost them more than their kernels on small inputs (encoding
// 26 000 points: 1.5 to 2.8 ms, 0.3 ms of it kernels).  Blocks come back only when no work that uses them is pending, so
// any thread and stream may take them next.  At most POOL_BYTES a device are kept (anything else is freed);
// ivf_free_index and an allocation of the library that fails give all of it back.
constexpr size_t POOL_BYTES = 1ull << 30;

struct DevPool {
    struct Block { void *p; size_t bytes; int dev; };
    static constexpr int MAX_IDLE = 64;                      // (a call has a dozen)
    std::mutex mu;
    Block idle[MAX_IDLE];                                     // oldest first; no containers: nothing here throws
    int n = 0;
    Block remove(int i)
    {
        const Block b = idle[i];
        for (--n; i < n; ++i) idle[i] = idle[i + 1];
        return b;
    }
    void trim(int dev)
    {
        Block out[MAX_IDLE];
        int m = 0;
        {
            std::lock_guard<std::mutex> lock(mu);
            for (int i = n - 1; i >= 0; --i)
                if (idle[i].dev == dev) out[m++] = remove(i);
        }
        for (int i = 0; i < m; ++i) (void)hipFree(out[i].p);
    }
    // a new allocation, here or for good; where there is no room for it the idle blocks of the device are given up first
    hipError_t fresh(void **p, size_t bytes)
    {
        *p = nullptr;
        hipError_t e = hipMalloc(p, bytes);
        if (e != hipErrorOutOfMemory) return e;
        (void)hipGetLastError();
        int dev = 0;
        if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
        trim(dev);
        if ((e = hipMalloc(p, bytes)) != hipSuccess) (void)hipGetLastError();   // (reported here, not by the next launch)
        return e;
    }
    // the smallest idle block that is not much larger than asked for, else a new one
    hipError_t take(void **p, size_t *got, int *dev, size_t bytes)
    {
        hipError_t e = hipGetDevice(dev);
        if (e != hipSuccess) return e;
        bytes = bytes < 4096 ? 4096 : bytes;
        {
            std::lock_guard<std::mutex> lock(mu);
            int best = -1;
            for (int i = 0; i < n; ++i)
                if (idle[i].dev == *dev && idle[i].bytes >= bytes && idle[i].bytes <= 2 * bytes && (best < 0 || idle[i].bytes < idle[best].bytes)) best = i;
            if (best >= 0) {
                const Block b = remove(best);
                *p = b.p;
                *got = b.bytes;
                return hipSuccess;
            }
        }
        *got = bytes;
        return fresh(p, bytes);
    }
    void give(void *p, size_t bytes, int dev)
    {
        if (bytes > POOL_BYTES) {
            (void)hipFree(p);
            return;
        }
        Block out[MAX_IDLE];                                  // what no longer fits, oldest first
        int m = 0;
        {
            std::lock_guard<std::mutex> lock(mu);
            if (n == MAX_IDLE) out[m++] = remove(0);
            size_t held = bytes;
            for (int i = 0; i < n; ++i)
                if (idle[i].dev == dev) held += idle[i].bytes;
            for (int i = 0; held > POOL_BYTES && i < n;)
                if (idle[i].dev == dev) {
                    held -= idle[i].bytes;
                    out[m++] = remove(i);
                } else {
                    ++i;
                }
            idle[n++] = Block{p, bytes, dev};
        }
        for (int i = 0; i < m; ++i) (void)hipFree(out[i].p);
    }
};

}  // namespace ivf
