// Device memory of the host side: blocks kept between calls.
#pragma once
#include <mutex>
#include <vector>

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
    std::mutex mu;
    std::vector<Block> idle;
    void trim(int dev)
    {
        std::vector<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu);
            for (size_t i = 0; i < idle.size();)
                if (idle[i].dev == dev) { out.push_back(idle[i]); idle[i] = idle.back(); idle.pop_back(); }
                else ++i;
        }
        for (const Block &b : out) (void)hipFree(b.p);
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
        return hipMalloc(p, bytes);
    }
    // the smallest idle block that is not much larger than asked for, else a new one
    hipError_t take(void **p, size_t *got, int *dev, size_t bytes)
    {
        hipError_t e = hipGetDevice(dev);
        if (e != hipSuccess) return e;
        bytes = bytes < 4096 ? 4096 : bytes;
        {
            std::lock_guard<std::mutex> lock(mu);
            size_t best = idle.size();
            for (size_t i = 0; i < idle.size(); ++i)
                if (idle[i].dev == *dev && idle[i].bytes >= bytes && idle[i].bytes <= 2 * bytes && (best == idle.size() || idle[i].bytes < idle[best].bytes)) best = i;
            if (best < idle.size()) {
                *p = idle[best].p;
                *got = idle[best].bytes;
                idle[best] = idle.back();
                idle.pop_back();
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
        std::vector<void *> out;                             // what no longer fits, oldest first
        {
            std::lock_guard<std::mutex> lock(mu);
            size_t held = bytes;
            idle.push_back(Block{p, bytes, dev});
            for (size_t i = 0; i + 1 < idle.size(); ++i)
                if (idle[i].dev == dev) held += idle[i].bytes;
            for (size_t i = 0; held > POOL_BYTES && i + 1 < idle.size();)
                if (idle[i].dev == dev) {
                    out.push_back(idle[i].p);
                    held -= idle[i].bytes;
                    idle.erase(idle.begin() + (long)i);
                } else {
                    ++i;
                }
        }
        for (void *q : out) (void)hipFree(q);
    }
};

}  // namespace ivf
