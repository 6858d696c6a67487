// Device memory of graphs and of their builds, kept for the next graph in processes that make
// graphs one after another.
//
// The driver wipes freed device memory before it hands it out again and hipMalloc waits for that:
// a program that creates, builds, walks and destroys a scale-20 graph of 31 M entries (4.2 GB a
// turn) took 10.7 ms a turn for the first 60 turns and 114 ms on average over 400, single
// hipMalloc calls up to 3 s; with blocks kept 8.8.
//
// Memory that is kept is memory that nothing else in the process, and no other process, can have.
// So a process that has not made a graph after destroying one keeps nothing: what it frees goes
// to the driver at once.  release() gives all back at any time and starts anew.
//
// Blocks of at least 1 MiB go to a list of idle blocks when they are freed, and a request takes
// the smallest idle block of its device that is at most 1/7 larger.  Bounds: 8 GiB and
// kIdleBlocks blocks per process, the oldest making room; blocks that kIdleTurns graphs in a row
// were destroyed without a use for go back to the driver, and all of a device's go back when
// hipMalloc fails.  A block is kept only when nothing on the device can use it any more.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <new>

namespace fw {

class DevPool {
public:
    hipError_t alloc(void **p, size_t bytes)
    {
        *p = nullptr;
        if (bytes < kMin) return fresh(p, bytes);
        int dev = 0;
        (void)hipGetDevice(&dev);
        bytes = (bytes + kMin - 1) / kMin * kMin;
        {
            std::lock_guard<std::mutex> lk(mu_);
            int best = -1;
            for (int i = 0; i < idle_n_; ++i)
                if (idle_[i].dev == dev && idle_[i].bytes >= bytes && idle_[i].bytes - bytes <= idle_[i].bytes / 8 &&
                    (best < 0 || idle_[i].bytes < idle_[best].bytes))
                    best = i;
            if (best >= 0 && live_n_ < kLive) {
                const Block b = take(best);
                live_[live_n_++] = b;
                *p = b.p;
                return hipSuccess;
            }
        }
        const hipError_t e = fresh(p, bytes);
        if (e != hipSuccess) return e;
        std::lock_guard<std::mutex> lk(mu_);
        if (live_n_ < kLive) live_[live_n_++] = Block{*p, bytes, dev, 0};  // (else freed to the driver)
        return hipSuccess;
    }

    // hipMalloc, with the idle blocks given back when it fails
    hipError_t fresh(void **p, size_t bytes)
    {
        hipError_t e = hipMalloc(p, bytes);
        int dev = 0;
        if (e != hipSuccess && hipGetDevice(&dev) == hipSuccess && give_back(dev)) {
            (void)hipGetLastError();
            e = hipMalloc(p, bytes);
        }
        if (e != hipSuccess) *p = nullptr;
        return e;
    }

    // unused: nothing on the device reads or writes the block any more
    void free(void *p, bool unused)
    {
        if (!p) return;
        Block out[kIdleBlocks + 1];
        int n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            Block b{p, 0, 0, turn_};
            for (int i = 0; i < live_n_; ++i)
                if (live_[i].p == p) {
                    b.bytes = live_[i].bytes;
                    b.dev = live_[i].dev;
                    live_[i] = live_[--live_n_];
                    break;
                }
            if (!unused || !keep_ || b.bytes == 0 || b.bytes > kMost) {
                out[n++] = b;
            } else {
                while (idle_n_ == kIdleBlocks || held_ + b.bytes > kMost) out[n++] = take(0);  // the oldest
                idle_[idle_n_++] = b;
                held_ += b.bytes;
            }
        }
        for (int i = 0; i < n; ++i) (void)hipFree(out[i].p);
    }

    // a graph is made
    void made()
    {
        std::lock_guard<std::mutex> lk(mu_);
        keep_ = keep_ || destroyed_;
    }

    // a graph was destroyed: blocks that nobody took for long go back
    void turn()
    {
        Block out[kIdleBlocks];
        int n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            destroyed_ = true;
            ++turn_;
            while (idle_n_ > 0 && turn_ - idle_[0].turn > kIdleTurns) out[n++] = take(0);
        }
        for (int i = 0; i < n; ++i) (void)hipFree(out[i].p);
    }

    // all idle blocks go back, and no more are kept until a graph is made after one destroyed from now on
    void release()
    {
        Block out[kIdleBlocks];
        int n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            keep_ = destroyed_ = false;
            while (idle_n_ > 0) out[n++] = take(idle_n_ - 1);
        }
        for (int i = 0; i < n; ++i) (void)hipFree(out[i].p);
    }

private:
    struct Block {
        void *p;
        size_t bytes;
        int dev;
        uint64_t turn;
    };
    static constexpr size_t kMin = (size_t)1 << 20, kMost = (size_t)8 << 30;
    static constexpr int kIdleBlocks = 64, kLive = 1024, kIdleTurns = 8;

    Block take(int i)  // (idle blocks stay in the order of their return)
    {
        const Block b = idle_[i];
        for (int k = i + 1; k < idle_n_; ++k) idle_[k - 1] = idle_[k];
        --idle_n_;
        held_ -= b.bytes;
        return b;
    }

    bool give_back(int dev)
    {
        Block out[kIdleBlocks];
        int n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (int i = 0; i < idle_n_;)
                if (idle_[i].dev == dev) out[n++] = take(i);
                else ++i;
        }
        for (int i = 0; i < n; ++i) (void)hipFree(out[i].p);
        return n > 0;
    }

    std::mutex mu_;
    Block idle_[kIdleBlocks], live_[kLive];
    int idle_n_ = 0, live_n_ = 0;
    size_t held_ = 0;
    uint64_t turn_ = 0;
    bool destroyed_ = false, keep_ = false;
};

// One per process; never destroyed, since graphs may outlive the library's statics.
inline DevPool &dev_pool()
{
    alignas(DevPool) static unsigned char at[sizeof(DevPool)];
    static DevPool *const pool = new (at) DevPool();
    return *pool;
}

// hipMalloc for what is not kept
template <typename P>
hipError_t dev_malloc(P **p, size_t bytes)
{
    void *v = nullptr;
    const hipError_t e = dev_pool().fresh(&v, bytes);
    *p = (P *)v;
    return e;
}

}  // namespace fw
