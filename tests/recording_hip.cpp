// Stands in for the HIP runtime under librh.so on a machine without a GPU: records which kernels are
// launched, counts allocations and synchronisations, and fails a chosen launch or host allocation.
// Nothing runs and device memory is only numbers.  Loaded before librh.so with RTLD_GLOBAL.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <map>
#include <new>
#include <string>

struct dim3 { uint32_t x, y, z; };
typedef int err_t;
enum { OK = 0, LAUNCH_FAILED = 719 };

static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::string g_log;
static int g_launches, g_mallocs, g_syncs, g_fail_launch = -1;
static err_t g_last;
static uint64_t g_next = 1ull << 40;
static int g_live;                                       // device allocations not yet freed
static void* g_pinned;
static std::atomic<long> g_fail_new{-1};
static struct { dim3 grid, block; size_t lds; void* stream; } g_cfg;

void* operator new(size_t n)
{
    if (g_fail_new >= 0 && g_fail_new.fetch_sub(1) == 0) throw std::bad_alloc();
    if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
void rec_reset() { g_log.clear(); g_launches = g_mallocs = g_syncs = 0; g_fail_launch = -1; g_last = OK; }
void rec_fail_launch(int k) { g_fail_launch = k; }       // the k-th launch from here on fails; -1: none
void rec_fail_new(long k) { g_fail_new = k; }             // likewise the k-th operator new of any thread
long rec_new_left() { return g_fail_new; }
int rec_mallocs() { return g_mallocs; }
int rec_live() { return g_live; }
void* rec_pinned() { return g_pinned; }                  // the host memory of the context created last
int rec_syncs() { return g_syncs; }
const char* rec_log() { return g_log.c_str(); }          // names of the launched kernels, one a line

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
err_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) { g_cfg = {grid, block, lds, stream}; return OK; }
err_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream)
{
    *grid = g_cfg.grid; *block = g_cfg.block; *lds = g_cfg.lds; *stream = g_cfg.stream;
    return OK;
}
err_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, void*)
{
    if (g_fail_launch >= 0 && g_fail_launch-- == 0) return g_last = LAUNCH_FAILED;
    g_log += names().at(f) + "\n";
    ++g_launches;
    return OK;
}
err_t hipGetLastError() { const err_t e = g_last; g_last = OK; return e; }
err_t hipMalloc(void** p, size_t n) { *p = (void*)g_next; g_next += (n + 4095) & ~(size_t)4095; ++g_mallocs; ++g_live; return OK; }
err_t hipFree(void* p) { if (p) --g_live; return OK; }
err_t hipHostMalloc(void** p, size_t n, unsigned) { *p = g_pinned = calloc(1, n); ++g_live; return *p ? OK : 2; }
err_t hipHostFree(void* p) { if (p) --g_live; if (p == g_pinned) g_pinned = nullptr; free(p); return OK; }
err_t hipMemcpy(void*, const void*, size_t, int) { return OK; }
err_t hipMemcpyAsync(void*, const void*, size_t, int, void*) { return OK; }
err_t hipMemset(void*, int, size_t) { return OK; }
err_t hipStreamSynchronize(void*) { ++g_syncs; return OK; }
err_t hipGetDevice(int* d) { *d = 0; return OK; }
err_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return OK; }
err_t hipFuncSetAttribute(const void*, int, int) { return OK; }
err_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)g_next; return OK; }
err_t hipEventCreate(void** e) { *e = (void*)1; return OK; }
err_t hipEventDestroy(void*) { return OK; }
err_t hipEventRecord(void*, void*) { return OK; }
err_t hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return OK; }
}
