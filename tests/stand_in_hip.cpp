// A stand-in for the HIP runtime that runs nothing: it notes which kernels libusl would launch, and refuses those a test names.  For host-side tests
// of what the library does around its launches; device memory is host memory that nobody reads.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

static std::map<const void*, std::string> kernels;
static std::string launched, refused;
static hipError_t last = hipSuccess;
static int allocated;
static bool capturing;

extern "C" {
const char* stand_in_launched() { return launched.c_str(); }   // names, one a line, since the last stand_in_start
void stand_in_start(const char* refuse) { launched.clear(); refused = refuse; allocated = 0; }
int stand_in_allocated() { return allocated; }   // calls of hipMalloc since then
void stand_in_capture(int on) { capturing = on != 0; }

void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) { *grid = *block = dim3(1); *lds = 0; *stream = nullptr; return hipSuccess; }
hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void**, size_t, hipStream_t) {
    const std::string name = kernels[fn];
    if (!refused.empty() && name.find(refused) != std::string::npos) return last = hipErrorLaunchFailure;
    launched += name + "\n";
    return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "refused by the stand-in"; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    memset(p, 0, sizeof *p);
    p->sharedMemPerBlock = 160 * 1024;
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { memset(a, 0, sizeof *a); a->numRegs = 64; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char place[1 << 16]; *p = place; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { ++allocated; *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemGetInfo(size_t* a, size_t* b) { *a = *b = (size_t)288 << 30; return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
}
