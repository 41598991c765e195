// Device-to-host copies into the caller's pageable memory.
//
// The runtime's own path copies a pageable destination chunk by chunk through one thread, which also
// takes the page faults of a freshly allocated array: 17 GB/s measured into arrays in use, 10 GB/s into the fresh
// 402 MB of a 4096^2 field output, on a link that moves 53 GB/s.  Here the device writes a ring of pinned
// chunks and a few threads, which live for the call alone, empty them into the destination.
#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>

#include "mcb_internal.h"

namespace mcb {
namespace {

// Chunks of 2 MB and four threads: fields of 1000 x 1200 (28.8 MB) 1.72 -> 0.99 ms into arrays in use, 2.8 -> 1.4
// into fresh ones, of 4096^2 23.7 -> 10.7 and 39 -> 11.2; fresh ones of 4096^2 with chunks of 1 MB 14.2 ms
// (each costs about 15 us besides its transfer), of 4 MB 11.1 but twice the pinned memory, with two
// threads 17.9 ms, with eight 12.1, against 12.5 in the same run.
constexpr int64_t CHUNK = int64_t(2) << 20;
constexpr int WORKERS = 4;

// The ring of pinned chunks (16 MB), one for the process: a lattice's copies are rare against its steps.  Used by
// one copy at a time (a copy that finds it taken goes the runtime's way), given back with the last context.
constexpr int R = 8;
std::mutex ring_mu;   // held for the length of a copy
char* ring = nullptr;
std::mutex count_mu;  // its own, held for no copy: contexts come and go while another thread's copy runs
int contexts = 0;

// Pinning takes 2 ms and a copy through the ring saves 25 us a megabyte into arrays in use, 50 into fresh ones:
// it is made once RING_AFTER bytes have been asked for in large copies, this one included, since there were
// contexts (made by the first large copy, it cost the first report of 800 x 700 nodes 2.9 ms instead of 1.3).
constexpr int64_t RING_AFTER = int64_t(48) << 20;
int64_t asked = 0;  // with ring_mu held

hipEvent_t ring_ev[R];
int ring_events = 0, ring_dev = -1;  // events belong to the device that was current when the ring was made

void ring_free() {
    while (ring_events > 0) (void)hipEventDestroy(ring_ev[--ring_events]);
    if (ring) (void)hipHostFree(ring);
    ring = nullptr;
}

bool ring_ready(int dev) {  // with ring_mu held
    // the context's device has to be current, for the events and for a null stream alike
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess || cur != dev) return false;
    if (ring) return dev == ring_dev;
    void* p = nullptr;
    hipError_t e = hipHostMalloc(&p, size_t(CHUNK * R), hipHostMallocDefault);
    if (e == hipSuccess) ring = static_cast<char*>(p);
    for (; e == hipSuccess && ring_events < R; ++ring_events) {
        e = hipEventCreateWithFlags(&ring_ev[ring_events], hipEventDisableTiming);
        if (e != hipSuccess) break;
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        ring_free();
        return false;
    }
    ring_dev = dev;
    return true;
}

hipError_t plain(mcb_ctx* c, void* dst, const void* src, int64_t n) {
    const hipError_t e = hipMemcpyAsync(dst, src, size_t(n), hipMemcpyDeviceToHost, c->stream);
    return e != hipSuccess ? e : hipStreamSynchronize(c->stream);
}

// Whether the runtime knows the destination.  Pinned memory it writes at the link's rate (28.8 MB 0.60 ms
// against 0.99 through the ring, 402 MB 7.8 against 10.7), and what is not plain host memory is its alone.
bool known(const void* dst) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, dst) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
}

// The ring's slot of chunk i is i % R.  A worker claims the next chunk, waits until it has arrived,
// copies it out and frees its slot; the calling thread issues the device copies, each into a freed
// slot, and marks the chunks that have arrived.  Every wait ends: a chunk arrives once its slot is
// freed by a worker that waits for nothing but earlier chunks, and an error ends all waits.
struct Transfer {
    std::mutex m;
    std::condition_variable arrived_cv, freed_cv;
    int64_t claimed = 0, arrived = 0, nch = 0;
    int64_t freed[R] = {};  // one past the last chunk copied out of each slot
    bool stop = false;

    void work(char* dst, int64_t n) {
        for (;;) {
            int64_t i;
            {
                std::unique_lock<std::mutex> l(m);
                if (claimed >= nch) return;
                i = claimed++;
                arrived_cv.wait(l, [&] { return arrived > i || stop; });
                if (arrived <= i) return;
            }
            std::memcpy(dst + i * CHUNK, ring + (i % R) * CHUNK, size_t(std::min(CHUNK, n - i * CHUNK)));
            {
                std::lock_guard<std::mutex> l(m);
                freed[i % R] = i + 1;
            }
            freed_cv.notify_one();
        }
    }
};

}  // namespace

hipError_t download(mcb_ctx* c, void* dst, const void* src, int64_t n) {
    // below 4 MB the runtime's copy is as fast as starting the threads
    if (n < (int64_t(4) << 20) || known(dst)) return plain(c, dst, src, n);
    std::unique_lock<std::mutex> mine(ring_mu, std::try_to_lock);
    if (!mine.owns_lock()) return plain(c, dst, src, n);
    asked += n;
    if (asked < RING_AFTER || !ring_ready(c->device)) {
        mine.unlock();
        return plain(c, dst, src, n);
    }
    Transfer t;
    t.nch = (n + CHUNK - 1) / CHUNK;
    std::thread th[WORKERS];
    int nth = 0;
    try {
        const int want = std::max(1, std::min(WORKERS, int(std::thread::hardware_concurrency()) / 2));
        for (; nth < want; ++nth) th[nth] = std::thread([&] { t.work(static_cast<char*>(dst), n); });
    } catch (...) {
        // as many as could be started
    }
    if (nth == 0) return plain(c, dst, src, n);
    hipError_t e = hipSuccess;
    int64_t issued = 0, seen = 0;
    while (seen < t.nch && e == hipSuccess) {
        bool room = false;
        if (issued < t.nch) {
            std::unique_lock<std::mutex> l(t.m);
            auto freed = [&] { return issued < R || t.freed[issued % R] == issued - R + 1; };
            if (seen == issued) t.freed_cv.wait(l, freed);  // nothing in flight: a worker frees the slot
            room = freed();
        }
        if (room) {
            const int k = int(issued % R);
            e = hipMemcpyAsync(ring + k * CHUNK, static_cast<const char*>(src) + issued * CHUNK,
                               size_t(std::min(CHUNK, n - issued * CHUNK)), hipMemcpyDeviceToHost, c->stream);
            if (e == hipSuccess) e = hipEventRecord(ring_ev[k], c->stream);
            ++issued;
        } else {
            e = hipEventSynchronize(ring_ev[seen % R]);
            if (e == hipSuccess) {
                ++seen;
                std::lock_guard<std::mutex> l(t.m);
                t.arrived = seen;
            }
            t.arrived_cv.notify_all();
        }
    }
    {
        std::lock_guard<std::mutex> l(t.m);
        t.stop = true;
    }
    t.arrived_cv.notify_all();
    for (int k = 0; k < nth; ++k) th[k].join();
    // after an error chunks may still be on their way into the ring: the next copy must not meet them, and
    // where the stream cannot be waited for either, none uses the ring again
    if (e != hipSuccess && hipStreamSynchronize(c->stream) != hipSuccess) ring_dev = -1;
    return e;
}

void download_open() {
    std::lock_guard<std::mutex> l(count_mu);
    ++contexts;
}

void download_close() {
    std::lock_guard<std::mutex> l(count_mu);
    if (--contexts > 0) return;
    std::lock_guard<std::mutex> r(ring_mu);  // free: a copy belongs to a context, and there is none
    ring_free();
    asked = 0;
}

}  // namespace mcb
