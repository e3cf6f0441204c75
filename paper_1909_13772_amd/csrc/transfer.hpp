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
#include <mutex>
#include <new>
#include <thread>

namespace wlb {

// Makes the device of a stream the current one: events have to be created on
// the device of the stream that records them, which need not be the caller's
// current one.
class OnDeviceOf {
public:
    explicit OnDeviceOf(hipStream_t st)
    {
        if (hipGetDevice(&before_) != hipSuccess || hipStreamGetDevice(st, &dev_) != hipSuccess) {
            (void)hipGetLastError();
            before_ = dev_ = -1;
        }
        if (dev_ != before_) (void)hipSetDevice(dev_);
    }
    ~OnDeviceOf()
    {
        if (dev_ != before_) (void)hipSetDevice(before_);
    }
    int device() const { return dev_; }

private:
    int before_ = -1, dev_ = -1;
};

// Pinned buffers of one transfer at a time, kept for the next one (PinnedPool).
class PinnedRing {
public:
    static constexpr int kSlots = 10;
    static constexpr size_t kChunk = (size_t)4 << 20;
    ~PinnedRing()
    {
        drop_events();
        if (base_) (void)hipHostFree(base_);
        if (small_) (void)hipHostFree(small_);
    }
    // At least n bytes for a transfer on `st`, n at most kSlots x kChunk; null
    // without pinned memory.  More than 1 MB is the whole ring: the runtime
    // takes 250 us for 2 to 10 MB, and 12 for 40 MB that it has had before.
    char *bytes(size_t n, hipStream_t st)
    {
        const OnDeviceOf on(st);
        if (n > n_) {
            if (base_) (void)hipHostFree(base_);
            n_ = n <= ((size_t)1 << 20) ? (n + 4095) & ~(size_t)4095 : kSlots * kChunk;
            base_ = pinned(n_);
            if (!base_) n_ = 0;
        }
        return static_cast<char *>(base_);
    }
    // Events of the device of `st`, one per slot; false without.
    bool events(hipStream_t st)
    {
        const OnDeviceOf on(st);
        if (on.device() != dev_) drop_events();
        dev_ = on.device();
        for (; n_ev_ < kSlots; ++n_ev_)
            if (hipEventCreateWithFlags(&ev_[n_ev_], hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                return false;
            }
        return true;
    }
    hipEvent_t event(int k) const { return ev_[k]; }
    // A few words that kernels write their sums to; null without pinned memory.
    double *sums(hipStream_t st)
    {
        if (!small_) {
            const OnDeviceOf on(st);
            small_ = pinned(4096);
        }
        return static_cast<double *>(small_);
    }

private:
    void drop_events()
    {
        for (; n_ev_ > 0; --n_ev_) (void)hipEventDestroy(ev_[n_ev_ - 1]);
    }
    static void *pinned(size_t n)
    {
        void *p = nullptr;
        if (hipHostMalloc(&p, n, hipHostMallocPortable) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    void *base_ = nullptr, *small_ = nullptr;
    size_t n_ = 0;
    hipEvent_t ev_[kSlots];
    int n_ev_ = 0, dev_ = -1;  // events, and the device they belong to
};

// The rings of the process that no transfer is using, at most kKeep (82 MB).
// Handles share them, so that pinned memory does not grow with the number of
// handles; concurrent transfers have a ring each.  All are given back with
// the last handle.
class PinnedPool {
public:
    static constexpr int kKeep = 2;
    static PinnedPool &process()
    {
        static PinnedPool p;
        return p;
    }
    // A handle counts as long as it has one of these.
    struct User {
        User() { process().users(1); }
        ~User() { process().users(-1); }
        User(const User &) = delete;
        User &operator=(const User &) = delete;
    };
    PinnedRing *take()
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (n_ > 0) return kept_[--n_];
        }
        return new (std::nothrow) PinnedRing;
    }
    void give(PinnedRing *r)
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (users_ > 0 && n_ < kKeep) {
                kept_[n_++] = r;
                r = nullptr;
            }
        }
        delete r;
    }

private:
    void users(int d)
    {
        PinnedRing *out[kKeep];
        int n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            users_ += d;
            if (users_ == 0)
                while (n_ > 0) out[n++] = kept_[--n_];
        }
        while (n > 0) delete out[--n];
    }
    std::mutex mu_;
    PinnedRing *kept_[kKeep] = {};
    int n_ = 0, users_ = 0;
};

// A ring for the transfers of one call on one stream, taken at its first use.
// The call is over when nothing on the stream uses the ring or the caller's
// arrays any more: after idle(), or after waiting for the stream where the call
// ended early.
class RingLease {
public:
    explicit RingLease(hipStream_t st) : st_(st) {}
    RingLease(const RingLease &) = delete;
    RingLease &operator=(const RingLease &) = delete;
    ~RingLease()
    {
        if (!idle_) (void)hipStreamSynchronize(st_);
        if (ring_) PinnedPool::process().give(ring_);
    }
    // Null where not even the object can be had.
    PinnedRing *get()
    {
        if (!ring_) ring_ = PinnedPool::process().take();
        busy();
        return ring_;
    }
    // Something that uses the ring or the caller's arrays is on the stream.
    void busy() { idle_ = false; }
    hipStream_t stream() const { return st_; }
    // The stream has been waited for since the last use.
    void idle() { idle_ = true; }

private:
    hipStream_t st_;
    PinnedRing *ring_ = nullptr;
    bool idle_ = true;
};

// One transfer of about `total` bytes in one direction on one stream, as any
// number of arrays.  An array goes over the link in pieces of up to 4 MB
// (45-54 GB/s; a piece costs some 9 us beyond its bytes, so small transfers
// take a quarter of their size), and a piece is copied on the host in parts
// of 512 KB by whichever thread is free.  Arrays in memory that the runtime
// knows are copied without buffers.  They are whole, like the others after
// flush(), once the stream has been waited for.  Device-side order is the
// stream's: a kernel launched before add() has finished when its pieces are
// read, and one launched after flush() sees every piece written.  Nothing here
// throws, for the C entry points that use it: its lists have a fixed size, and
// threads that cannot be had are done without.
class HostCopy {
public:
    static constexpr size_t kMinToHost = (size_t)4 << 20, kMinToDevice = (size_t)128 << 20;
    HostCopy(RingLease &lease, bool to_host, size_t total) : lease_(lease), to_host_(to_host), st_(lease.stream())
    {
        // a smaller transfer is over before buffers and threads have paid for
        // themselves, at 25 GB/s from pageable memory and some 15 into it (us
        // by the runtime's own copy / through the buffers: density of 48^3, 0.9
        // MB, 64 / 113, of 64^3, 2.1 MB, 143 / 170, of 80^3, 4.1 MB, 246 / 225)
        if (total < (to_host ? kMinToHost : kMinToDevice)) return;
        chunk_ = std::min(PinnedRing::kChunk, std::max<size_t>((size_t)256 << 10, total / 4));
        chunk_ = (chunk_ + 4095) & ~(size_t)4095;
        ring_ = lease.get();
        base_ = ring_ ? ring_->bytes(chunk_ * PinnedRing::kSlots, st_) : nullptr;
        pinned_ = base_ && ring_->events(st_);
        if (!pinned_) return;
        cpu_set_t cs;
        const int cpus = sched_getaffinity(0, sizeof cs, &cs) == 0 ? CPU_COUNT(&cs) : 1;
        want_ = std::min((int)std::min<size_t>(kWorkers, total >> 20), cpus - 1);  // one more thread per MB
    }
    ~HostCopy()
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            done_ = true;
        }
        cv_.notify_all();
        for (int k = 0; k < n_workers_; ++k) workers_[k].join();
    }
    // Whether pageable arrays go through the pinned buffers.
    bool buffered() const { return pinned_; }
    // Memory the runtime knows (pinned or registered by the caller, managed,
    // device): the copy engine reads and writes it itself.
    static bool mapped(const void *p)
    {
        hipPointerAttribute_t a;
        if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
        (void)hipGetLastError();
        return false;
    }
    hipError_t add(void *host, void *dev, size_t n)
    {
        // through the buffers pinned arrays would only be slower (populations
        // of 100^3, 152 MB: 3.7 ms against 3.2; density of 64^3: 163 us against 64)
        lease_.busy();
        if (!pinned_ || mapped(host))
            return to_host_ ? hipMemcpyAsync(host, dev, n, hipMemcpyDeviceToHost, st_)
                            : hipMemcpyAsync(dev, host, n, hipMemcpyHostToDevice, st_);
        for (size_t o = 0; o < n; o += chunk_) {
            const int k = next_;
            next_ = (next_ + 1) % PinnedRing::kSlots;
            if (!free_slot(k)) return err_;
            const size_t m = std::min(chunk_, n - o);
            if (to_host_) {
                hipError_t e = hipMemcpyAsync(slot(k), static_cast<char *>(dev) + o, m, hipMemcpyDeviceToHost, st_);
                if (e == hipSuccess) e = hipEventRecord(ring_->event(k), st_);
                if (e != hipSuccess) return e;
            }
            {
                std::lock_guard<std::mutex> lk(mu_);
                piece_[k] = Piece{static_cast<char *>(dev) + o, m, (int)((m + kPart - 1) / kPart), true, false};
                for (size_t q = 0; q < m; q += kPart)
                    queue_[(head_ + n_queued_++) % kParts] = Part{static_cast<char *>(host) + o + q, q, std::min(kPart, m - q), k};
            }
            cv_.notify_all();
            // threads start while the link is busy with what is under way
            if (n_workers_ < want_) spawn();
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
    static constexpr size_t kPart = (size_t)512 << 10;
    static constexpr int kWorkers = 7, kParts = PinnedRing::kSlots * (int)(PinnedRing::kChunk / kPart);
    struct Piece {
        char *dev;
        size_t n;
        int left;  // parts not yet copied
        bool busy;
        bool ready;  // to the device: all parts copied, not yet enqueued
    };
    struct Part {
        char *host;
        size_t off, n;
        int slot;
    };
    void spawn()
    {
        try {
            workers_[n_workers_] = std::thread([this] {
                std::unique_lock<std::mutex> lk(mu_);
                for (;;) {
                    cv_.wait(lk, [this] { return done_ || n_queued_ > 0; });
                    if (n_queued_ == 0) return;
                    run_one(lk);
                }
            });
            ++n_workers_;
        } catch (...) {
            want_ = 0;  // the threads there are and the caller's own do the rest
        }
    }
    // Waits until slot k holds no unfinished piece, working on parts and
    // enqueuing finished ones meanwhile; false after an error.
    bool free_slot(int k)
    {
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            if (ready_ > 0)
                send_ready(lk);
            else if (!piece_[k].busy)
                return err_ == hipSuccess;
            else if (n_queued_ > 0)
                run_one(lk);
            else
                cv_.wait(lk);
        }
    }
    // Enqueues the pieces that are whole in their buffers.  Only the thread
    // that makes the transfer does this: the stream may be the calling
    // thread's own (hipStreamPerThread), another one in a copying thread.
    void send_ready(std::unique_lock<std::mutex> &lk)
    {
        for (int k = 0; k < PinnedRing::kSlots; ++k) {
            Piece &w = piece_[k];
            if (!w.ready) continue;
            w.ready = false;
            --ready_;
            if (err_ == hipSuccess) {
                lk.unlock();
                hipError_t e = hipMemcpyAsync(w.dev, slot(k), w.n, hipMemcpyHostToDevice, st_);
                if (e == hipSuccess) e = hipEventRecord(ring_->event(k), st_);
                lk.lock();
                if (e != hipSuccess && err_ == hipSuccess) err_ = e;
            }
            w.busy = false;
        }
    }
    // Takes the oldest part and copies it with the lock released.
    void run_one(std::unique_lock<std::mutex> &lk)
    {
        const Part p = queue_[head_];
        head_ = (head_ + 1) % kParts;
        --n_queued_;
        lk.unlock();
        hipError_t e;
        if (to_host_) {
            populate(p.host, p.n);
            e = hipEventSynchronize(ring_->event(p.slot));
            if (e == hipSuccess) std::memcpy(p.host, slot(p.slot) + p.off, p.n);
        } else {
            // the buffer's previous piece may still be on its way to the device
            e = hipEventSynchronize(ring_->event(p.slot));
            if (e == hipSuccess) std::memcpy(slot(p.slot) + p.off, p.host, p.n);
        }
        lk.lock();
        if (e != hipSuccess && err_ == hipSuccess) err_ = e;
        Piece &w = piece_[p.slot];
        if (--w.left > 0) return;
        if (to_host_) {
            w.busy = false;
        } else {
            w.ready = true;
            ++ready_;
        }
        cv_.notify_all();
    }
    // Maps the pages of a destination in one call: 9 GB/s per thread of 4 KiB
    // pages against 5 when the copy faults them in one by one.
    static void populate(char *host, size_t n)
    {
        const uintptr_t a = reinterpret_cast<uintptr_t>(host) & ~(uintptr_t)4095;
        const uintptr_t b = (reinterpret_cast<uintptr_t>(host) + n + 4095) & ~(uintptr_t)4095;
        constexpr int kPopulateWrite = 23;  // MADV_POPULATE_WRITE; unknown to older kernels, then it does nothing
        (void)madvise(reinterpret_cast<void *>(a), b - a, kPopulateWrite);
    }

    char *slot(int k) const { return base_ + (size_t)k * chunk_; }

    RingLease &lease_;
    PinnedRing *ring_ = nullptr;
    char *base_ = nullptr;
    const bool to_host_;
    hipStream_t st_;
    size_t chunk_ = 0;
    bool pinned_ = false;
    int want_ = 0;
    std::mutex mu_;
    std::condition_variable cv_;
    Part queue_[kParts];  // parts of the busy pieces not yet taken, oldest at head_
    int head_ = 0, n_queued_ = 0;
    Piece piece_[PinnedRing::kSlots] = {};
    bool done_ = false;
    int next_ = 0, ready_ = 0;
    hipError_t err_ = hipSuccess;
    std::thread workers_[kWorkers];
    int n_workers_ = 0;
};

}  // namespace wlb
