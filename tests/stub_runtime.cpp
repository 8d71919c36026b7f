// A HIP runtime without a device for CPU tests of the library's host side: allocations are
// counted, kernels are not run, and like the real runtime it keeps the last error of a thread
// until hipGetLastError reads it. Loaded with global symbols before libcwo.so, its functions
// are the ones the library binds to.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <mutex>

namespace {
std::mutex mu;
std::map<void*, size_t> blocks;
size_t held = 0, refuse = 0;  // allocations of `refuse` bytes and more fail (0: none)
bool recording = false;       // some stream of the process records a graph
int allocations_recording = 0;
thread_local int last = 0, capture_mode = 0;  // mode 2: relaxed
struct Dim {
    unsigned x, y, z;
};
struct {
    Dim grid, block;
    size_t shmem;
    void* stream;
} config;
}  // namespace

extern "C" {
size_t stub_held() { return held; }
void stub_refuse(size_t bytes) { refuse = bytes; }
void stub_record(int on) { recording = on; }
int stub_unsafe_allocations() { return allocations_recording; }

int hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> g(mu);
    if (recording && capture_mode != 2) {
        ++allocations_recording;
        return last = 900;  // hipErrorStreamCaptureUnsupported, and the capture is lost
    }
    if (refuse && n >= refuse) return last = 2;  // hipErrorOutOfMemory
    *p = std::malloc(1);
    blocks[*p] = n;
    held += n;
    return 0;
}
int hipFree(void* p) {
    std::lock_guard<std::mutex> g(mu);
    auto it = blocks.find(p);
    if (it == blocks.end()) return p ? last = 1 : 0;
    held -= it->second;
    blocks.erase(it);
    std::free(p);
    return 0;
}
int hipGetLastError() {
    const int e = last;
    last = 0;
    return e;
}
int hipThreadExchangeStreamCaptureMode(int* mode) {
    const int was = capture_mode;
    capture_mode = *mode;
    *mode = was;
    return 0;
}
int hipStreamIsCapturing(void*, int* status) { return *status = 0; }
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { return 0; }
int hipExtLaunchKernel(const void*, Dim, Dim, void**, size_t, void*, void*, void*, int) { return 0; }
int __hipPushCallConfiguration(Dim g, Dim b, size_t shmem, void* stream) {
    config = {g, b, shmem, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* shmem, void** stream) {
    *g = config.grid, *b = config.block, *shmem = config.shmem, *stream = config.stream;
    return 0;
}
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int hipGetSymbolAddress(void** p, const void*) {
    static char array[8];
    *p = array;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* v, const void*, int, size_t) { return *v = 2, 0; }
int hipGetDevice(int* d) { return *d = 0; }
int hipGetDeviceCount(int* n) { return *n = 1, 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = std::malloc(1), 0; }
int hipStreamDestroy(void* s) { return std::free(s), 0; }
int hipEventCreate(void** e) { return *e = std::malloc(1), 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return *e = std::malloc(1), 0; }
int hipEventDestroy(void* e) { return std::free(e), 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventQuery(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 1.0f, 0; }
}
