// csrc/download.hip built for the host against the stand-in runtime, and what the tests set and read.
#include "download.hip"

static mcb_ctx g_ctx[2];

extern "C" {
void t_open(int k, int device) {
    g_ctx[k].device = device;
    mcb::download_open();
}
void t_close() { mcb::download_close(); }
int t_download(int k, void* dst, const void* src, int64_t n) { return mcb::download(&g_ctx[k], dst, src, n); }
void t_reset(int device, int fail_record_at, int fail_sync) {
    std::lock_guard<std::mutex> l(fake::m);
    fake::issued.clear();
    fake::device = device;
    fake::records = fake::syncs = 0;
    fake::fail_record_at = fail_record_at;
    fake::fail_sync = fail_sync;
}
int64_t t_in_flight() {
    std::lock_guard<std::mutex> l(fake::m);
    return int64_t(fake::queue.size());
}
void t_drop() {  // forget what is in flight
    std::lock_guard<std::mutex> l(fake::m);
    fake::queue.clear();
    fake::marks.clear();
}
// copies since the last reset that went to the ring
int64_t t_ring_copies() {
    std::lock_guard<std::mutex> l(fake::m);
    int64_t k = 0;
    for (auto& c : fake::issued) {
        const char* d = static_cast<const char*>(c.dst);
        const char* r = static_cast<const char*>(fake::ring);
        k += r && d >= r && d < r + fake::ring_bytes;
    }
    return k;
}
int t_ring_there() { return fake::ring != nullptr; }
void t_hold(int on) {
    std::lock_guard<std::mutex> l(fake::m);
    fake::hold = on != 0;
    fake::held = false;
    fake::cv.notify_all();
}
void t_wait_held() {
    std::unique_lock<std::mutex> l(fake::m);
    fake::cv.wait(l, [] { return fake::held; });
}
void t_register(const void* p, int type) {
    fake::reg_ptr = p;
    fake::reg_type = hipMemoryType(type);
}
}
