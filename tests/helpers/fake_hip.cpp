// Stand-in for the HIP runtime, preloaded before libgwg.so: device memory is a
// budget of bytes, copies do nothing (from the device: zeros), kernel launches
// are written to a log.  For tests of what the library's host side allocates
// and launches, on a machine without a GPU and with as little memory as a test
// wants.
#define __HIP_PLATFORM_AMD__
#include <cstdio>
#include <cstring>
#include <dlfcn.h>
#include <map>
#include <string>

#include <hip/hip_runtime_api.h>

#include "gwg_internal.h"

namespace {
std::map<char*, size_t> g_mem;
size_t g_used = 0, g_total = (size_t)288 << 30, g_refuse_lo = 1, g_refuse_hi = 0;
char* g_next = (char*)0x100000000000;
bool g_capture = false;
std::string g_log, g_sizes, g_asked;
double g_clock = 0.0;                      // ms of the launches so far
std::map<void*, double> g_event;
double g_cost64 = 1.0, g_cost128 = 1.0, g_cost256 = 1.0;
struct Call { dim3 grid, block; size_t smem; hipStream_t stream; } g_call;
const char* kernel_name(const void* f)
{
    Dl_info di;
    return dladdr(f, &di) && di.dli_sname ? di.dli_sname : "?";
}
}  // namespace

extern "C" {
// control
void fake_memory(size_t total) { g_total = total; }
void fake_refuse(size_t lo, size_t hi) { g_refuse_lo = lo; g_refuse_hi = hi; }   // allocations of these sizes fail
size_t fake_used() { return g_used; }
void fake_capture(int on) { g_capture = on != 0; }
void fake_costs(double c64, double c128, double c256) { g_cost64 = c64; g_cost128 = c128; g_cost256 = c256; }
const char* fake_log() { return g_log.c_str(); }
const char* fake_asked() { return g_asked.c_str(); }       // kernels whose occupancy was asked for
const char* fake_sizes() { return g_sizes.c_str(); }       // of every allocation asked for
void fake_clear() { g_log.clear(); g_sizes.clear(); }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n)
{
    *p = nullptr;
    g_sizes += std::to_string(n) + "\n";
    if (g_used + n > g_total || (n >= g_refuse_lo && n <= g_refuse_hi)) return hipErrorOutOfMemory;
    g_mem[g_next] = n;
    g_used += n;
    *p = g_next;
    g_next += (n + 4095) / 4096 * 4096;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    const auto it = g_mem.find((char*)p);
    if (it != g_mem.end()) { g_used -= it->second; g_mem.erase(it); }
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = g_total - g_used; *t = g_total; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void*, size_t n, hipMemcpyKind k)
{
    if (k == hipMemcpyDeviceToHost) std::memset(d, 0, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipStreamSynchronize(hipStream_t) { g_log += "wait\n"; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(g_next += 64); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { g_event[(void*)e] = g_clock; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(g_event[(void*)b] - g_event[(void*)a]);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = g_next; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int wg, size_t)
{
    g_asked += std::string(kernel_name(f)) + "\n";
    *n = 512 / wg;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sm, hipStream_t s) { g_call = { g, b, sm, s }; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sm, hipStream_t* s)
{
    *g = g_call.grid; *b = g_call.block; *sm = g_call.smem; *s = g_call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t sm, hipStream_t)
{
    const char* name = kernel_name(f);
    char line[768];
    std::snprintf(line, sizeof(line), "%s %u %u", name, g.x * g.y * g.z, b.x);
    g_log += line;
    if (std::strstr(name, "k_trace_fwd") || std::strstr(name, "k_omega_grad") || std::strstr(name, "k_trace_bwd")) {
        const gwg::SceneDev* s = (const gwg::SceneDev*)args[0];
        std::snprintf(line, sizeof(line), " items=%lld rays=%lld pool=%d memo=%d dirs=%p", (long long)s->n_items,
                      (long long)s->rays_per_tile, s->pool, s->memo, (const void*)s->dirs);
        g_log += line;
        if (std::strstr(name, "k_trace_fwd")) {
            const gwg::AdjStore* a = (const gwg::AdjStore*)args[8];
            std::snprintf(line, sizeof(line), " regions=%lld ck_regions=%lld ck_nb=%d ck_evan=%d",
                          (long long)(s->n_items * a->waves), (long long)a->ck_regions, a->ck_nb, a->ck_evan);
            g_log += line;
        }
        if (std::strstr(name, "k_trace_fwd")) g_clock += b.x == 64 ? g_cost64 : b.x == 128 ? g_cost128 : g_cost256;
    }
    g_log += "\n";
    return hipSuccess;
}
}
