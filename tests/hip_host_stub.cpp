// Stand-ins for the HIP runtime calls that the distance makes, for CPU tests of its locking: the "device" is a
// property of the calling thread, kernels are not run, the wait for a stream returns when as many threads wait at
// once as were announced, or after five seconds, and a launch can be held up until another thread records an event, or half a second.
// Loaded with global symbols in front of the library.
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <mutex>

typedef int err;
static thread_local int device = 0;
static std::mutex mu;
static std::condition_variable cv;
static int expected = 1, waiting = 0, met = 0;
static bool hold = false, in_launch = false, launched = false, early = false;

extern "C" {
void stub_expect(int threads) {
    std::lock_guard<std::mutex> lock(mu);
    expected = threads;
    waiting = met = 0;
}
void stub_device(int d) { device = d; }
int stub_met() { return met; }   // waits that found all the others waiting
void stub_hold_launch() { hold = true; }                          // the next one
void stub_wait_for_launch() {
    std::unique_lock<std::mutex> lock(mu);
    cv.wait(lock, [] { return in_launch; });
}
int stub_early() { return early; }   // an event was recorded while the launch that it is to stand behind was not made yet

err hipGetDevice(int* d) { *d = device; return 0; }
err hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
err hipDeviceSynchronize() { return 0; }
err hipMalloc(void** p, size_t n) { *p = std::malloc(n); return 0; }
err hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return 0; }
err hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
err hipEventCreateWithFlags(void** e, unsigned) { *e = nullptr; return 0; }
err hipStreamIsCapturing(void*, int* s) { *s = 0; return 0; }
err hipGetLastError() { return 0; }
err hipEventRecord(void*, void*) {
    std::lock_guard<std::mutex> lock(mu);
    if (in_launch && !launched) early = true;
    cv.notify_all();
    return 0;
}
err hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
err hipLaunchKernel(const void*, unsigned long long, unsigned, unsigned long long, unsigned, void**, size_t, void*) {
    std::unique_lock<std::mutex> lock(mu);
    if (!hold) return 0;
    hold = false;
    in_launch = true;
    cv.notify_all();
    cv.wait_for(lock, std::chrono::milliseconds(500), [] { return early; });
    launched = true;
    return 0;
}
struct Dim { unsigned x, y, z; };
err __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
err __hipPopCallConfiguration(Dim* g, Dim* b, size_t* s, void** st) { *g = *b = Dim{1, 1, 1}; *s = 0; *st = nullptr; return 0; }
err hipStreamSynchronize(void*) {
    std::unique_lock<std::mutex> lock(mu);
    ++waiting;
    cv.notify_all();
    if (cv.wait_for(lock, std::chrono::seconds(5), [] { return waiting >= expected; })) ++met;
    return 0;
}
}
