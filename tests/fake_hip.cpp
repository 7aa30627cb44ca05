// A HIP runtime of host memory for tests of libfbp's host code without a GPU: allocations
// come from malloc and can be made to fail by size, a launch is written down (kernel name,
// workgroups) and not run.  Loaded before libfbp with global symbols, it answers every HIP
// call the library makes.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string kernel;
    long long blocks;
};
std::map<const void*, std::string> names;
std::vector<Launch> launches;
size_t fail_from = SIZE_MAX;       // allocations of this many bytes or more fail
size_t allocated = 0;              // bytes, since the last reset
int last_error = 0, capturing = 0;
int device_word = 0;
int fail(int e) {
    last_error = e;
    return e;
}
}  // namespace

struct dim3_abi {
    uint32_t x, y, z;
};

extern "C" {

void fake_reset() {
    launches.clear();
    allocated = 0;
    last_error = 0;
}
void fake_fail_from(size_t bytes) { fail_from = bytes; }
void fake_capturing(int on) { capturing = on; }
size_t fake_allocated() { return allocated; }
int fake_launches() { return (int)launches.size(); }
const char* fake_kernel(int i) { return launches[(size_t)i].kernel.c_str(); }
long long fake_blocks(int i) { return launches[(size_t)i].blocks; }

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPopCallConfiguration(void*, void*, size_t*, void*) { return 0; }

int hipMalloc(void** p, size_t n) {
    if (n >= fail_from) {
        *p = nullptr;
        return fail(2);                                     // hipErrorOutOfMemory
    }
    allocated += n;
    *p = std::malloc(n ? n : 1);
    return 0;
}
int hipFree(void* p) {
    std::free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n ? n : 1);
    return 0;
}
int hipHostFree(void* p) {
    std::free(p);
    return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) {
    std::memset(d, v, n);
    return 0;
}
int hipLaunchKernel(const void* f, dim3_abi grid, dim3_abi, void**, size_t, void*) {
    launches.push_back({names[f], (long long)grid.x * grid.y * grid.z});
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 1;
    return 0;
}
int hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = 256;
    return 0;
}
int hipGetDevicePropertiesR0600(void*, int) { return fail(1); }
int hipGetSymbolAddress(void** p, const void*) {
    *p = &device_word;
    return 0;
}
const char* hipGetErrorName(int) { return "fake error"; }
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipPeekAtLastError() { return last_error; }
int hipEventCreate(void** e) {
    *e = &device_word;
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) {
    *e = &device_word;
    return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) {
    *t = 1.0f;
    return 0;
}
int hipEventQuery(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) {
    *s = &device_word;
    return 0;
}
int hipStreamIsCapturing(void*, int* status) {
    *status = capturing;
    return 0;
}
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) {
    *g = &device_word;
    return 0;
}
int hipGraphInstantiate(void** g, void*, void*, char*, size_t) {
    *g = &device_word;
    return 0;
}
int hipGraphDestroy(void*) { return 0; }
int hipGraphLaunch(void*, void*) { return 0; }

}  // extern "C"
