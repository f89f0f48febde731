// A stand-in for the HIP runtime on a machine without a GPU: device memory is
// host memory (zeros), kernels do nothing, and every request is written down.
// Loaded ahead of libmsz.so, its functions take the place of the runtime's, so
// that the host side of the library can be tested on its own: where scratch
// comes from, what happens when memory is short, what grids are launched.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::map<void*, size_t> live;
std::vector<void*> pinned;
std::string text;
size_t largest = ~size_t(0);  // a larger request of device memory fails
int current = 0, of_stream = 0;
unsigned word = 0;     // what copies of four bytes to the host bring
bool pattern = false;  // copies to the host bring 0, 1, 0, 1, ... as floats
hipError_t last = hipSuccess;

hipError_t result(hipError_t e) {  // the last error stays until it is asked for
    if (e != hipSuccess) last = e;
    return e;
}
hipError_t take(void** p, size_t bytes, const std::string& from) {
    const bool fails = from != "host" && bytes > largest;
    text += from + " " + std::to_string(bytes) + (fails ? " fails\n" : "\n");
    if (fails) return result(hipErrorOutOfMemory);
    void* q = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED) return result(hipErrorOutOfMemory);
    live[q] = bytes;
    *p = q;
    return hipSuccess;
}
dim3 pushed_grid, pushed_block;
size_t pushed_shared;
hipStream_t pushed_stream;
}  // namespace

extern "C" {

void fake_set(size_t largest_request, int current_device, int device_of_streams) {
    largest = largest_request;
    current = current_device;
    of_stream = device_of_streams;
    text.clear();
}
void fake_word(unsigned w) { word = w; }
void fake_pattern(int on) { pattern = on != 0; }
const char* fake_log() { return text.c_str(); }
size_t fake_live_bytes() {
    size_t n = 0;
    for (const auto& b : live) n += b.second;
    return n;
}

hipError_t hipGetDevice(int* dev) { return *dev = current, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* dev) { return *dev = of_stream, hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) { return take(p, bytes, "device"); }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    const hipError_t e = take(p, bytes, "host");
    if (e == hipSuccess) pinned.push_back(*p);
    return e;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
    const auto it = live.find(p);
    if (it == live.end()) return result(hipErrorInvalidValue);
    munmap(p, it->second);
    live.erase(it);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t) {
    std::memcpy(dst, src, bytes);
    if (kind == hipMemcpyDeviceToHost && bytes == 4) std::memcpy(dst, &word, 4);
    for (size_t i = 0; pattern && kind == hipMemcpyDeviceToHost && i < bytes / 4; ++i)
        static_cast<float*>(dst)[i] = static_cast<float>(i & 1);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t bytes, hipStream_t) {
    std::memset(dst, v, bytes);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

// The rest of what a correction needs.  A graph is its list of launches; once
// launched, the first word of every pinned allocation is cleared, which ends
// the loop of a correction (its results are zeros).
hipError_t hipMalloc(void** p, size_t bytes) { return take(p, bytes, "device"); }
hipError_t hipFree(void* p) { return hipFreeAsync(p, nullptr); }
hipError_t hipHostGetDevicePointer(void** dev, void* host, unsigned) { return *dev = host, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 4, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    return *s = reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(4096)), hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = nullptr, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t* g, unsigned) {
    return *g = reinterpret_cast<hipGraph_t>(new std::string), hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t*, hipGraph_t g, const hipGraphNode_t*, size_t,
                                 const hipKernelNodeParams* p) {
    *reinterpret_cast<std::string*>(g) += "step " + std::to_string(p->gridDim.x) + "\n";
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    return *e = reinterpret_cast<hipGraphExec_t>(g), hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    text += *reinterpret_cast<std::string*>(e);
    for (void* p : pinned) std::memset(p, 0, 4);
    return hipSuccess;
}

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
    pushed_grid = grid, pushed_block = block, pushed_shared = shared, pushed_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
    *grid = pushed_grid, *block = pushed_block, *shared = pushed_shared, *s = pushed_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
    text += "launch " + std::to_string(grid.x) + " " + std::to_string(block.x) + "\n";
    // (the runtime takes fewer than 2^32 threads)
    return static_cast<unsigned long long>(grid.x) * block.x >= 1ull << 32 ? result(hipErrorInvalidConfiguration)
                                                                           : hipSuccess;
}

}  // extern "C"
