// Device blocks kept from one object or call for the next.
//
// A pair of 300 x 300 x 640 float32 scans takes some twenty blocks, about 1 GB together
// (two more volumes where the inputs are on the host), and gives them back
// when it is destroyed.  hipFree waits for the device and then costs 0.27 ms a
// large block, and memory given back to the driver is cleared before it is
// given out again: a program that creates one pair after another runs at the
// clearing rate once the device's memory has been through it.  Kept blocks cost
// neither: that pair, its evaluation at the coarser levels and its end take
// 0.65 ms instead of 5.0 ms at first and 42 ms in the long run (1.24 ms before the
// ingest was one kernel a level).
//
// One cache per device, shared by the contexts on it and by the objects that
// hold blocks of it, and emptied with the last of them.  Only idle blocks come
// here: their owner has waited for the stream (or the device) that last used
// them, so any stream of any thread can take them.  The idle blocks are bounded
// (1 / 32 of the device's memory, 64 host blocks); the oldest are freed beyond
// that, and all of them when an allocation fails, which is then tried again, or
// when the caller asks for it (octmc_trim).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <deque>
#include <memory>
#include <mutex>
#include <vector>

namespace octmc {

struct Block {
    void* p = nullptr;
    size_t bytes = 0;
};

class BlockCache {
public:
    // the cache of `device`, which is current
    static std::shared_ptr<BlockCache> of(int device)
    {
        constexpr int kMax = 64;
        static std::mutex mu;
        static std::weak_ptr<BlockCache> all[kMax];
        if (device < 0 || device >= kMax) return std::make_shared<BlockCache>();
        std::lock_guard<std::mutex> lk(mu);
        std::shared_ptr<BlockCache> c = all[device].lock();
        if (!c) all[device] = c = std::make_shared<BlockCache>();
        return c;
    }

    BlockCache()
    {
        size_t avail = 0, total = 0;
        if (hipMemGetInfo(&avail, &total) == hipSuccess) cap_ = total / 32;
    }
    ~BlockCache() { trim(); }
    BlockCache(const BlockCache&) = delete;
    BlockCache& operator=(const BlockCache&) = delete;

    // a block of at least `bytes` on the current device (the cache's), or null and the reason
    Block take(size_t bytes, hipError_t* err)
    {
        bytes = (bytes + kGrain - 1) / kGrain * kGrain;
        if (!bytes) bytes = kGrain;
        {
            std::lock_guard<std::mutex> lk(mu_);
            auto best = idle_.end();
            for (auto it = idle_.begin(); it != idle_.end(); ++it)
                if (it->bytes >= bytes && it->bytes - bytes <= bytes / 8 &&
                    (best == idle_.end() || it->bytes < best->bytes))
                    best = it;
            if (best != idle_.end()) {
                const Block b = *best;
                idle_.erase(best);
                held_ -= b.bytes;
                return b;
            }
        }
        Block b{nullptr, bytes};
        *err = hipMalloc(&b.p, bytes);
        if (*err == hipSuccess) return b;
        if (*err == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            trim();
            *err = hipMalloc(&b.p, bytes);
            if (*err == hipSuccess) return b;
        }
        return Block{};
    }

    // an idle block back
    void give(Block b)
    {
        std::vector<Block> out;
        try {
            std::lock_guard<std::mutex> lk(mu_);
            if (b.bytes <= cap_) {
                idle_.push_back(b);
                held_ += b.bytes;
                b.p = nullptr;
                while (held_ > cap_ || idle_.size() > kMaxIdle) {
                    out.push_back(idle_.front());
                    held_ -= idle_.front().bytes;
                    idle_.pop_front();
                }
            }
        } catch (const std::bad_alloc&) {
        }
        if (b.p) (void)hipFree(b.p);
        for (const Block& q : out) (void)hipFree(q.p);
    }

    // pinned host memory of kHostBytes, or null and the reason
    void* take_host(hipError_t* err)
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (!host_.empty()) {
                void* p = host_.back();
                host_.pop_back();
                return p;
            }
        }
        void* p = nullptr;
        *err = hipHostMalloc(&p, kHostBytes, hipHostMallocDefault);
        return *err == hipSuccess ? p : nullptr;
    }
    void give_host(void* p)
    {
        try {
            std::lock_guard<std::mutex> lk(mu_);
            if (host_.size() < kMaxHost) {
                host_.push_back(p);
                p = nullptr;
            }
        } catch (const std::bad_alloc&) {
        }
        if (p) (void)hipHostFree(p);
    }

    // gives every idle block back to the driver
    void trim()
    {
        std::deque<Block> dev;
        std::vector<void*> host;
        {
            std::lock_guard<std::mutex> lk(mu_);
            dev.swap(idle_);
            host.swap(host_);
            held_ = 0;
        }
        for (const Block& b : dev) (void)hipFree(b.p);
        for (void* p : host) (void)hipHostFree(p);
    }

    static constexpr size_t kHostBytes = 4096;

private:
    static constexpr size_t kGrain = 4096;  // the allocator's own
    static constexpr size_t kMaxIdle = 1024, kMaxHost = 64;
    std::mutex mu_;
    std::deque<Block> idle_;  // oldest first
    std::vector<void*> host_;
    size_t cap_ = 0, held_ = 0;
};

// The blocks of one object or call.  They go back to the cache if their owner
// has said that nothing uses them any more (settle, or `idle` after a wait for
// the device); otherwise, as on the way out of an error, hipFree waits for the
// device first.
struct Blocks {
    std::shared_ptr<BlockCache> cache;
    std::vector<Block> dev;
    std::vector<void*> host;
    bool idle = false;
    hipError_t err = hipErrorInvalidValue;  // of the last get that gave nothing

    explicit Blocks(std::shared_ptr<BlockCache> c = nullptr) : cache(std::move(c)) {}
    Blocks(const Blocks&) = delete;
    Blocks& operator=(const Blocks&) = delete;
    ~Blocks()
    {
        for (const Block& b : dev) {
            if (idle)
                cache->give(b);
            else
                (void)hipFree(b.p);
        }
        for (void* p : host) {
            if (idle)
                cache->give_host(p);
            else
                (void)hipHostFree(p);
        }
    }
    void* get(size_t bytes)
    {
        idle = false;
        dev.reserve(dev.size() + 1);
        const Block b = cache->take(bytes, &err);
        if (b.p) dev.push_back(b);
        return b.p;
    }
    // pinned host memory for `n` float64 (at most kHostBytes)
    double* get_host(size_t n)
    {
        if (n * 8 > BlockCache::kHostBytes) return nullptr;
        idle = false;
        host.reserve(host.size() + 1);
        void* p = cache->take_host(&err);
        if (p) host.push_back(p);
        return static_cast<double*>(p);
    }
    // waits for the stream that used the blocks last
    hipError_t settle(hipStream_t s)
    {
        const hipError_t e = hipStreamSynchronize(s);
        idle = e == hipSuccess;
        return e;
    }
};

}  // namespace octmc
