// Host transfers (transfer.hpp) on the CPU, against stand-ins for the runtime
// calls they make: "device" memory is host memory, copies are done at once,
// and each stand-in checks how it is called.  One check per command-line name.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <new>
#include <thread>

#include "transfer.hpp"

static void bad(const char *what)
{
    fprintf(stderr, "%s\n", what);
    exit(1);
}

static std::atomic<bool> no_memory{false};
void *operator new(size_t n)
{
    void *p = no_memory ? nullptr : malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

// memory known to the runtime
static char *known = nullptr;
static size_t known_bytes = 0;
static int fail_after = -1;  // copies that succeed before one fails (-1: all)
static bool is_known(const void *p) { return known && (const char *)p >= known && (const char *)p < known + known_bytes; }

static std::atomic<int> n_copies{0}, n_known{0}, n_pinned{0}, n_alive{0}, n_waits{0};
static const std::thread::id main_thread = std::this_thread::get_id();

// two devices; a stream's handle is 1000 times its device (0: the null stream)
static thread_local int device = 0;
static int device_of(hipStream_t st) { return st ? (int)((uintptr_t)st / 1000) : device; }
struct Event {
    int device;
};

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t st, hipDevice_t *d) { return *d = device_of(st), hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return ++n_pinned, ++n_alive, (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { return --n_alive, free(p), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return ++n_waits, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)malloc(sizeof(Event)), ((Event *)*e)->device = device, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
// a copying thread is delayed now and then, so that pieces end out of order
hipError_t hipEventSynchronize(hipEvent_t)
{
    static std::atomic<unsigned> k{0};
    if (++k % 5 == 0) std::this_thread::sleep_for(std::chrono::microseconds(50));
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    if (((Event *)e)->device != device_of(st)) return hipErrorInvalidHandle;
    if (std::this_thread::get_id() != main_thread) bad("an event is recorded by a copying thread");
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    memset(a, 0, sizeof *a);
    a->type = is_known(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t)
{
    if (fail_after >= 0 && fail_after-- == 0) return hipErrorUnknown;
    n_known += is_known(kind == hipMemcpyDeviceToHost ? dst : src);
    if (std::this_thread::get_id() != main_thread) bad("a copy is enqueued by a copying thread");
    ++n_copies;
    return memcpy(dst, src, n), hipSuccess;
}
}

using namespace wlb;

// Arrays of sizes around the pieces and parts, in both directions and through
// one ring, arrive whole.
static void round_trips(hipStream_t st)
{
    const size_t mb = (size_t)1 << 20;
    const size_t sizes[] = {1, 4095, 512 << 10, (512 << 10) + 1, 4 * mb - 8, 4 * mb, 4 * mb + 1, 63 * mb + 5};
    for (int k = 0; k < 4; ++k)
        for (bool to_host : {true, false}) {
            RingLease lease(st);
            HostCopy c(lease, to_host, 140 * mb);
            char *src[8], *dst[8];
            for (int i = 0; i < 8; ++i) {
                src[i] = (char *)malloc(sizes[i]);
                dst[i] = (char *)malloc(sizes[i]);
                for (size_t o = 0; o < sizes[i]; o += 97) src[i][o] = (char)(o * 31 + i + k);
                memset(dst[i], 0x55, sizes[i]);
                if (c.add(to_host ? dst[i] : src[i], to_host ? src[i] : dst[i], sizes[i]) != hipSuccess) bad("add");
                if (i == 4 && c.flush() != hipSuccess) bad("flush");
            }
            if (c.flush() != hipSuccess) bad("flush");
            lease.idle();
            for (int i = 0; i < 8; ++i) {
                if (memcmp(src[i], dst[i], sizes[i])) bad("contents");
                free(src[i]);
                free(dst[i]);
            }
        }
}

// An array that the runtime knows is copied as a whole from or to its place,
// whatever the others of the transfer are.
static void known_memory()
{
    const size_t n = ((size_t)9 << 20) + 3;
    char *dev = (char *)malloc(n), *other = (char *)malloc(n);
    known = (char *)calloc(n, 1);
    known_bytes = n;
    for (bool to_host : {true, false}) {
        n_copies = n_known = 0;
        memset(to_host ? dev : known, to_host ? 1 : 2, n);
        RingLease lease(nullptr);
        HostCopy c(lease, to_host, (size_t)140 << 20);
        if (c.add(known, dev, n) != hipSuccess || c.flush() != hipSuccess) bad("add");
        if (n_copies != 1 || n_known != 1) bad("a known array is copied through buffers");
        if (memcmp(known, dev, n)) bad("contents");
        if (c.add(other, dev, n) != hipSuccess || c.flush() != hipSuccess) bad("add");
        if (n_copies != 4 || n_known != 1) bad("an ordinary array is not copied through buffers");
        if (memcmp(other, dev, n)) bad("contents");
    }
}

// A transfer to the host below kMinToHost is left to the runtime: one copy
// per array, to its place, and no buffers.
static void small_transfers()
{
    for (size_t n : {(size_t)885 * 1000, HostCopy::kMinToHost - 1, HostCopy::kMinToHost}) {
        char *dev = (char *)malloc(n), *host = (char *)calloc(n, 1);
        memset(dev, 3, n);
        known = nullptr;
        n_copies = n_pinned = 0;
        {
            RingLease lease(nullptr);
            HostCopy c(lease, true, n);
            if (c.add(host, dev, n) != hipSuccess || c.flush() != hipSuccess) bad("add");
        }
        if (memcmp(host, dev, n)) bad("contents");
        const bool small = n < HostCopy::kMinToHost;
        if (small ? n_copies != 1 || n_pinned != 0 : n_pinned == 0) bad(small ? "a small transfer takes buffers" : "no buffers");
        free(dev);
        free(host);
    }
}

// The pinned buffers of the process: kept between transfers and shared by the
// handles, one for each transfer under way, bounded, and gone with the last
// handle.
static void pool()
{
    const size_t n = (size_t)20 << 20;
    auto use = [&](RingLease &l) {
        char *p = l.get()->bytes(n, nullptr);
        if (!p || !l.get()->sums(nullptr)) bad("no buffer");
        return p;
    };
    PinnedPool::User *a = new PinnedPool::User, *b = new PinnedPool::User;
    if (n_pinned != 0) bad("pinned memory before the first transfer");
    char *first;
    {
        RingLease l(nullptr);
        first = use(l);
        l.idle();
    }
    if (n_waits != 0) bad("waited for an idle stream");
    {
        RingLease l(nullptr);
        if (use(l) != first) bad("the buffer is not kept");
    }
    if (n_waits != 1) bad("given back without waiting for the stream");
    if (n_pinned != 2) bad("more than one buffer for transfers in turn");
    {
        RingLease l[5] = {RingLease(nullptr), RingLease(nullptr), RingLease(nullptr), RingLease(nullptr), RingLease(nullptr)};
        char *p[5];
        for (int k = 0; k < 5; ++k) {
            p[k] = use(l[k]);
            for (int j = 0; j < k; ++j)
                if (p[j] == p[k]) bad("two transfers share a buffer");
        }
    }
    if (n_alive != 2 * PinnedPool::kKeep) bad("the kept buffers are not bounded");
    delete a;
    if (n_alive == 0) bad("a handle that is left lost the buffers");
    RingLease late(nullptr);
    use(late);
    delete b;
    if (n_alive != 2) bad("buffers outlive the last handle");
}

// A call that ends early waits for the stream: copies from and to the
// caller's arrays may still be under way.
static void early_end()
{
    const size_t n = (size_t)1 << 20;
    char *dev = (char *)malloc(n);
    known = (char *)calloc(n, 1);
    known_bytes = n;
    for (size_t total : {n, (size_t)200 << 20})
        for (bool to_host : {true, false}) {
            n_waits = 0;
            fail_after = 1;
            {
                RingLease lease(nullptr);
                HostCopy c(lease, to_host, total);
                if (c.add(known, dev, n) != hipSuccess) bad("add");
                if (c.add(known, dev, n) == hipSuccess) bad("a failed copy is not reported");
            }
            if (n_waits != 1) bad("returned while a copy may be under way");
        }
    n_waits = 0;
    {
        RingLease lease(nullptr);
    }
    if (n_waits != 0) bad("waited for nothing");
}

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "pool")) {
        pool();  // ends with a transfer that outlives its handle
        if (n_alive != 0) bad("buffers are left");
        puts("ok");
        return 0;
    }
    PinnedPool::User handle;
    if (!strcmp(what, "round_trips")) round_trips(nullptr);
    else if (!strcmp(what, "no_memory")) {
        no_memory = true;
        round_trips(nullptr);
    }
    else if (!strcmp(what, "devices")) {
        for (int d : {1, 0, 1}) {
            round_trips((hipStream_t)(uintptr_t)(1000 * d + 1));
            if (device != 0) bad("the caller's device has changed");
        }
    }
    else if (!strcmp(what, "known_memory")) known_memory();
    else if (!strcmp(what, "small_transfers")) small_transfers();
    else if (!strcmp(what, "early_end")) early_end();
    else bad("unknown check");
    puts("ok");
}
