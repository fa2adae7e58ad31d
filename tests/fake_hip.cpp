// The HIP entry points that the library calls, for tests of its host code on a machine without a GPU: device memory is host memory, as
// much as fake_limit allows, copies are made at once and launches do nothing but count.  Preloaded in front of the real runtime.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

static size_t limit_bytes = (size_t)1 << 40, used_bytes, n_launches, n_null_copies;
static std::map<void*, size_t>& live() { static std::map<void*, size_t> m; return m; }
static int last_error;
enum { OK = 0, OUT_OF_MEMORY = 2 };

extern "C" {
void fake_limit(size_t bytes) { limit_bytes = bytes; }
size_t fake_used() { return used_bytes; }
size_t fake_launches() { return n_launches; }
size_t fake_null_copies() { return n_null_copies; }          // copies and fills on the null stream

int hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (n > limit_bytes - used_bytes) return last_error = OUT_OF_MEMORY;
    *p = malloc(n);
    live()[*p] = n;
    used_bytes += n;
    return OK;
}
int hipFree(void* p) {
    auto it = live().find(p);
    if (it == live().end()) { fprintf(stderr, "hipFree of what hipMalloc did not give\n"); abort(); }
    used_bytes -= it->second;
    live().erase(it);
    free(p);
    return OK;
}
int hipMemGetInfo(size_t* free_bytes, size_t* total) { *free_bytes = limit_bytes - used_bytes; *total = limit_bytes; return OK; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return OK; }
int hipHostFree(void* p) { free(p); return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int) { n_null_copies++; memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* st) { n_null_copies += !st; memcpy(d, s, n); return OK; }
int hipMemset(void* d, int v, size_t n) { n_null_copies++; memset(d, v, n); return OK; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { n_null_copies += !st; memset(d, v, n); return OK; }
int hipGetLastError() { const int e = last_error; last_error = OK; return e; }
const char* hipGetErrorString(int) { return "fake"; }
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipGetDeviceCount(int* d) { *d = 1; return OK; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return OK; }
int hipDeviceSynchronize() { return OK; }
static int give(void** p) { *p = malloc(8); return OK; }
static int take(void* p) { free(p); return OK; }
int hipEventCreate(void** e) { return give(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return give(e); }
int hipEventDestroy(void* e) { return take(e); }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return OK; }
int hipEventRecord(void*, void*) { return OK; }
int hipStreamCreateWithFlags(void** s, unsigned) { return give(s); }
int hipExtStreamCreateWithCUMask(void** s, uint32_t, const uint32_t*) { return give(s); }
int hipStreamDestroy(void* s) { return take(s); }
int hipStreamSynchronize(void*) { return OK; }
int hipStreamWaitEvent(void*, void*, unsigned) { return OK; }
int hipStreamBeginCapture(void*, int) { return OK; }
int hipStreamEndCapture(void*, void** g) { return give(g); }
int hipGraphDestroy(void* g) { return take(g); }
int hipGraphInstantiate(void** e, void*, void*, void*, size_t) { return hipMalloc(e, 1 << 20); }
int hipGraphExecDestroy(void* e) { return hipFree(e); }
int hipGraphLaunch(void*, void*) { return OK; }
int hipFuncSetAttribute(const void*, int, int) { return OK; }
int hipLaunchKernel(const void*, ...) { n_launches++; return last_error; }
int hipExtLaunchKernel(const void*, ...) { n_launches++; return last_error; }
static char array[(32 << 20)];
int hipGetSymbolAddress(void** p, const void*) { *p = array; return OK; }
void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(...) {}
void __hipRegisterVar(...) {}
}
