// transfer.hpp -- copies between caller-owned host arrays and the device
// through a ring of pinned buffers, with the host-side copy (and the first
// touch of fresh destination pages) spread over a few threads.
//
// Why: an asynchronous copy to pageable memory ran at 9.7 GB/s (fields of a
// 320^3 run, 1.05 GB: 105 ms), bound by one thread that faults the caller's
// pages in and copies.  On the same host pinned copies reach 45-56 GB/s in
// pieces of 2-32 MB, and copying into untouched pages 15 GB/s per thread
// (huge pages) or 5 GB/s (4 KiB pages; 9 GB/s when populated first), 57-89
// GB/s with 4-8 threads: with the pieces in flight on several threads the
// link is what bounds the transfer.
#pragma once

#include <hip/hip_runtime.h>
#include <sched.h>
#include <stdint.h>
#include <sys/mman.h>

#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace wlb {

// Pinned buffers of one handle, allocated at its first transfer and released
// with it (kSlots x kChunk = 40 MB at most).
class PinnedRing {
public:
    static constexpr int kSlots = 10;
    static constexpr size_t kChunk = (size_t)4 << 20;
    ~PinnedRing()
    {
        for (hipEvent_t e : ev_) (void)hipEventDestroy(e);
        if (base_) (void)hipHostFree(base_);
    }
    // Room for kSlots pieces of `chunk` bytes; false without pinned memory.
    bool reserve(size_t chunk)
    {
        if (chunk > chunk_) {
            if (base_) (void)hipHostFree(base_);
            base_ = nullptr;
            chunk_ = 0;
            if (hipHostMalloc(&base_, chunk * kSlots, hipHostMallocDefault) != hipSuccess) {
                (void)hipGetLastError();
                base_ = nullptr;
                return false;
            }
            chunk_ = chunk;
        }
        while ((int)ev_.size() < kSlots) {
            hipEvent_t e;
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                return false;
            }
            ev_.push_back(e);
        }
        return true;
    }
    char *slot(int k) const { return static_cast<char *>(base_) + (size_t)k * chunk_; }
    hipEvent_t event(int k) const { return ev_[k]; }

private:
    void *base_ = nullptr;
    size_t chunk_ = 0;
    std::vector<hipEvent_t> ev_;
};

// One transfer of about `total` bytes in one direction on one stream, as any
// number of pieces.  Device-side order is the stream's: a kernel launched
// before add() has finished when its pieces are read, and one launched after
// flush() sees every piece written.
class HostCopy {
public:
    HostCopy(PinnedRing &ring, bool to_host, hipStream_t st, size_t total) : ring_(ring), to_host_(to_host), st_(st)
    {
        // pieces small enough that copying one overlaps the transfer of the
        // next also where the whole transfer is small
        chunk_ = std::min(PinnedRing::kChunk, std::max<size_t>((size_t)256 << 10, total / 16));
        chunk_ = (chunk_ + 4095) & ~(size_t)4095;
        pinned_ = ring.reserve(chunk_);
        if (!pinned_) return;
        cpu_set_t cs;
        const int cpus = sched_getaffinity(0, sizeof cs, &cs) == 0 ? CPU_COUNT(&cs) : 1;
        const int want = (int)std::min<size_t>(7, total / ((size_t)3 << 19));  // one more thread per 1.5 MB
        int dev = 0;
        (void)hipGetDevice(&dev);
        try {
            for (int k = 0; k < std::min(want, cpus - 1); ++k)
                workers_.emplace_back([this, dev] {
                    (void)hipSetDevice(dev);
                    work();
                });
        } catch (const std::system_error &) {
            // fewer threads: the caller's own does the rest
        }
    }
    ~HostCopy()
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            done_ = true;
        }
        cv_.notify_all();
        for (std::thread &t : workers_) t.join();
    }
    hipError_t add(void *host, void *dev, size_t n)
    {
        if (!pinned_) {
            const hipError_t e = to_host_ ? hipMemcpyAsync(host, dev, n, hipMemcpyDeviceToHost, st_)
                                          : hipMemcpyAsync(dev, host, n, hipMemcpyHostToDevice, st_);
            return e;
        }
        for (size_t o = 0; o < n; o += chunk_) {
            Job j{static_cast<char *>(host) + o, static_cast<char *>(dev) + o, std::min(chunk_, n - o), next_};
            next_ = (next_ + 1) % PinnedRing::kSlots;
            if (!free_slot(j.slot)) return err_;
            if (to_host_) {
                hipError_t e = hipMemcpyAsync(ring_.slot(j.slot), j.dev, j.n, hipMemcpyDeviceToHost, st_);
                if (e == hipSuccess) e = hipEventRecord(ring_.event(j.slot), st_);
                if (e != hipSuccess) return e;
            }
            {
                std::lock_guard<std::mutex> lk(mu_);
                busy_[j.slot] = true;
                queue_.push_back(j);
            }
            cv_.notify_one();
        }
        return hipSuccess;
    }
    // Every piece added so far is in the host array (to_host) or enqueued on
    // the stream (to the device).
    hipError_t flush()
    {
        if (!pinned_) return hipSuccess;
        for (int k = 0; k < PinnedRing::kSlots; ++k)
            if (!free_slot(k)) return err_;
        return err_;
    }

private:
    struct Job {
        char *host, *dev;
        size_t n;
        int slot;
    };
    // Waits until slot k holds no unfinished piece, working on pieces
    // meanwhile; false after an error.
    bool free_slot(int k)
    {
        std::unique_lock<std::mutex> lk(mu_);
        while (busy_[k]) {
            if (!queue_.empty())
                run_one(lk);
            else
                cv_.wait(lk);
        }
        return err_ == hipSuccess;
    }
    void work()
    {
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            cv_.wait(lk, [this] { return done_ || !queue_.empty(); });
            if (queue_.empty()) return;
            run_one(lk);
        }
    }
    // Takes the oldest piece and copies it with the lock released.
    void run_one(std::unique_lock<std::mutex> &lk)
    {
        const Job j = queue_.front();
        queue_.pop_front();
        lk.unlock();
        const hipError_t e = to_host_ ? to_host(j) : to_device(j);
        lk.lock();
        if (e != hipSuccess && err_ == hipSuccess) err_ = e;
        busy_[j.slot] = false;
        cv_.notify_all();
    }
    hipError_t to_host(const Job &j)
    {
        const uintptr_t a = reinterpret_cast<uintptr_t>(j.host) & ~(uintptr_t)4095;
        const uintptr_t b = (reinterpret_cast<uintptr_t>(j.host) + j.n + 4095) & ~(uintptr_t)4095;
        constexpr int kPopulateWrite = 23;  // MADV_POPULATE_WRITE; unknown to older kernels, then it does nothing
        (void)madvise(reinterpret_cast<void *>(a), b - a, kPopulateWrite);
        const hipError_t e = hipEventSynchronize(ring_.event(j.slot));
        if (e == hipSuccess) std::memcpy(j.host, ring_.slot(j.slot), j.n);
        return e;
    }
    hipError_t to_device(const Job &j)
    {
        // the buffer's previous piece may still be on its way to the device
        hipError_t e = hipEventSynchronize(ring_.event(j.slot));
        if (e != hipSuccess) return e;
        std::memcpy(ring_.slot(j.slot), j.host, j.n);
        e = hipMemcpyAsync(j.dev, ring_.slot(j.slot), j.n, hipMemcpyHostToDevice, st_);
        return e == hipSuccess ? hipEventRecord(ring_.event(j.slot), st_) : e;
    }

    PinnedRing &ring_;
    const bool to_host_;
    hipStream_t st_;
    size_t chunk_ = 0;
    bool pinned_ = false;
    std::mutex mu_;
    std::condition_variable cv_;
    std::deque<Job> queue_;
    bool busy_[PinnedRing::kSlots] = {};
    bool done_ = false;
    int next_ = 0;
    hipError_t err_ = hipSuccess;
    std::vector<std::thread> workers_;
};

}  // namespace wlb
