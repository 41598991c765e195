// A host-only stand-in for the few runtime calls of csrc/download.hip, so that its host logic (errors, waits,
// locks) is tested without a GPU.  Copies are held back until something waits for them, as on a device;
// a test can make a call fail, hold the waits, and read what is still in flight.
#pragma once
#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#define __constant__

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorUnknown = 999 };
typedef void* hipStream_t;
typedef int* hipEvent_t;
enum hipMemcpyKind { hipMemcpyDeviceToHost = 2 };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2, hipMemoryTypeManaged = 3 };
struct hipPointerAttribute_t {
    hipMemoryType type;
};

namespace fake {
struct Copy {
    void* dst;
    const void* src;
    size_t n;
};
inline std::mutex m;
inline std::condition_variable cv;
inline std::vector<Copy> queue;       // issued, not yet landed
inline std::vector<Copy> issued;      // every copy since the last reset
inline std::vector<std::pair<int*, size_t>> marks;
inline std::vector<int*> events;
inline int device = 0, fail_record_at = -1, fail_sync = 0, records = 0, syncs = 0;
inline bool hold = false, held = false;
inline void* ring = nullptr;          // the one pinned allocation
inline size_t ring_bytes = 0;
inline const void* reg_ptr = nullptr; // a pointer the runtime knows, and as what
inline hipMemoryType reg_type = hipMemoryTypeUnregistered;

inline void land(size_t k) {  // the first k copies arrive
    for (size_t i = 0; i < k; ++i) std::memcpy(queue[i].dst, queue[i].src, queue[i].n);
    queue.erase(queue.begin(), queue.begin() + long(k));
    for (auto& e : marks) e.second = e.second > k ? e.second - k : 0;
}
}  // namespace fake

inline const char* hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) {
    *d = fake::device;
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    fake::ring = *p;
    fake::ring_bytes = n;
    return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
    std::free(p);
    fake::ring = nullptr;
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = new int(0);
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::lock_guard<std::mutex> l(fake::m);
    fake::queue.push_back({d, s, n});
    fake::issued.push_back({d, s, n});
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    std::lock_guard<std::mutex> l(fake::m);
    if (fake::records++ == fake::fail_record_at) return hipErrorUnknown;
    for (auto& k : fake::marks)
        if (k.first == e) {
            k.second = fake::queue.size();
            return hipSuccess;
        }
    fake::marks.push_back({e, fake::queue.size()});
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    std::unique_lock<std::mutex> l(fake::m);
    fake::held = fake::hold;
    fake::cv.notify_all();
    fake::cv.wait(l, [] { return !fake::hold; });
    for (auto& k : fake::marks)
        if (k.first == e) fake::land(k.second);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) {
    std::unique_lock<std::mutex> l(fake::m);
    ++fake::syncs;
    if (fake::fail_sync) return hipErrorUnknown;
    fake::cv.wait(l, [] { return !fake::hold; });
    fake::land(fake::queue.size());
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    if (fake::reg_ptr && p == fake::reg_ptr) {
        a->type = fake::reg_type;
        return hipSuccess;
    }
    return hipErrorInvalidValue;
}
