// The part of the HIP runtime that libivfadcr calls, on host memory and without kernels: a launch does nothing.  It lets the host code of
// the library - what it allocates, frees and reports, and what it does when an allocation fails - run without a GPU.  Loaded into a
// process of its own, in front of the library.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>

struct Dim { uint32_t x, y, z; };

static std::map<void*, size_t> live;
static size_t live_bytes;
static long fail_at = -1;   // allocations until one fails (-1: none does)
static long n_attributes, n_launches;
static struct { Dim grid, block; size_t lds; void* stream; } call;

extern "C" {
void host_fail_allocation(long n) { fail_at = n; }
size_t host_live_bytes() { return live_bytes; }
long host_attributes() { return n_attributes; }
long host_launches() { return n_launches; }

int hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (fail_at >= 0 && fail_at-- == 0) return 2;   // out of memory
    *p = malloc(n ? n : 1);
    live[*p] = n;
    live_bytes += n;
    return *p ? 0 : 2;
}
int hipFree(void* p) {
    if (!p) return 0;
    if (!live.count(p)) abort();   // given back twice, or never taken
    live_bytes -= live[p];
    live.erase(p);
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemGetInfo(size_t* a, size_t* b) { *a = *b = (size_t)1 << 38; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { memset(d, v, n); return 0; }
int hipFuncSetAttribute(const void*, int, int) { ++n_attributes; return 0; }
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { ++n_launches; return 0; }
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* st) { call = {g, b, lds, st}; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** st) { *g = call.grid; *b = call.block; *lds = call.lds; *st = call.stream; return 0; }
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int hipGetSymbolAddress(void** p, const void*) { static char byte; *p = &byte; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }   // (the library then takes its default number of compute units)
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
int hipPointerGetAttributes(void*, const void*) { return 1; }   // memory of the host
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }
}
