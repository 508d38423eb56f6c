// A HIP runtime that records what it is asked for and does nothing, for looking at the library's host side without a
// GPU: loaded before liblgc.so with global symbols, its functions are the ones that the library finds.  Device memory is
// a range of addresses that nobody reads; launches and allocations go to a log.
#include <hip/hip_runtime_api.h>

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

namespace {
std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> k; return k; }
std::string log_text, taken;
uintptr_t next_address = 1ull << 44;
unsigned char static_array[64];
std::map<uintptr_t, size_t> &held() { static std::map<uintptr_t, size_t> h; return h; }   // device memory: address, bytes
const void *shares[4];   // the first pointers of the last encoder launch's first argument: input, output, sums, counts

hipError_t record_launch(const void *f, dim3 grid) {
    char dims[64];
    snprintf(dims, sizeof dims, " %u %u %u\n", grid.x, grid.y, grid.z);
    log_text += "launch " + kernels()[f] + dims;
    return hipSuccess;
}
}  // namespace

extern "C" {
// the log since the last call of this function
const char *recorded() { taken.swap(log_text); log_text.clear(); return taken.c_str(); }

void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
static dim3 call_grid, call_block;
static size_t call_lds;
static hipStream_t call_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) { call_grid = g; call_block = b; call_lds = l; call_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) { *g = call_grid; *b = call_block; *l = call_lds; *s = call_stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t) {
    if (kernels()[f].find("k_encoder_fused") != std::string::npos) memcpy(shares, args[0], sizeof shares);
    return record_launch(f, grid);
}
// where the last encoder launch's blocks meet, and the device memory from `at` on that is still allocated
const void *encoder_shares(int counts) { return shares[2 + counts]; }
size_t allocated_from(uintptr_t at) {
    auto next = held().upper_bound(at);
    if (next == held().begin()) return 0;
    --next;
    return at < next->first + next->second ? next->first + next->second - at : 0;
}
hipError_t hipExtLaunchKernel(const void *f, dim3 grid, dim3, void **, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) { return record_launch(f, grid); }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }   // (the header gives the name its version)
hipError_t hipDeviceGetAttribute(int *x, hipDeviceAttribute_t, int) { *x = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
int capturing;   // whether the stream is being recorded; negative: the runtime refuses to say
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    if (capturing < 0) return hipErrorStreamCaptureImplicit;
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
    *p = (void *)next_address;
    held()[next_address] = bytes;
    next_address += (bytes + 8191) / 4096 * 4096;
    log_text += "malloc " + std::to_string(bytes) + "\n";
    return hipSuccess;
}
hipError_t hipFree(void *p) { held().erase((uintptr_t)p); return hipSuccess; }
void *pinned;   // the last pinned allocation
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { *p = pinned = calloc(1, bytes); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = static_array; return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpy(void *to, const void *, size_t bytes, hipMemcpyKind kind) { if (kind == hipMemcpyDeviceToHost) memset(to, 0, bytes); return hipSuccess; }
}
