// A stand-in for the HIP runtime under the host code of libtlb: memory is host memory, kernels are recorded and
// not run, and chosen calls can be made to fail.  Built and loaded by standin.py in a process of its own, before
// the library, so that the library's calls find it first.
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

struct dim3_ {
    uint32_t x, y, z;
};

namespace {
struct Launch {
    std::string name;
    const void* first[2];  // the first two pointers of the kernel's argument block (source and destination buffer)
    uint32_t grid, block;
};
std::vector<Launch> launches;
std::map<const void*, std::string> names;
std::map<std::string, double> cost;  // ms of a launch whose name contains the key
double now = 0.0;                    // ms of the launches so far
int last_error = 0, fail_launch = -1, fail_malloc = -1, capturing = 0;
dim3_ cfg_grid, cfg_block;
constexpr int kOutOfMemory = 2, kInvalidValue = 1;

int sticky(int e)
{
    if (e) last_error = e;
    return e;
}
int allocate(void** p, size_t n)
{
    if (fail_malloc >= 0 && fail_malloc-- == 0) return sticky(kOutOfMemory);
    *p = malloc(n ? n : 1);
    return *p ? 0 : sticky(kOutOfMemory);
}
}  // namespace

extern "C" {
// ---- control ----
void standin_clear() { launches.clear(); }
int standin_count() { return (int)launches.size(); }
const char* standin_name(int i) { return launches[i].name.c_str(); }
const void* standin_pointer(int i, int k) { return launches[i].first[k]; }
uint32_t standin_grid(int i) { return launches[i].grid; }
void standin_fail_launch(int after) { fail_launch = after; }  // the launch after so many fails, once
void standin_fail_malloc(int after) { fail_malloc = after; }
void standin_capturing(int on) { capturing = on; }
void standin_cost(const char* part, double ms) { cost[part] = ms; }

// ---- kernels ----
void** __hipRegisterFatBinary(const void*)
{
    static void* module;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*)
{
    int st = 0;
    char* s = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    names[host] = s ? s : device;
    free(s);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t, void*)
{
    cfg_grid = grid;
    cfg_block = block;
    return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* shared, void** stream)
{
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = 0;
    *stream = nullptr;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_ grid, dim3_ block, void** args, size_t, void*)
{
    if (fail_launch >= 0 && fail_launch-- == 0) return sticky(kInvalidValue);
    Launch l;
    l.name = names.count(f) ? names[f] : "?";
    memcpy(l.first, args[0], l.name.find("Args") != std::string::npos ? sizeof(l.first) : 0);
    l.grid = grid.x;
    l.block = block.x;
    for (const auto& c : cost)
        if (l.name.find(c.first) != std::string::npos) now += c.second;
    launches.push_back(l);
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, 0; }
int hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return e;
}

// ---- device, memory ----
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, 0; }
int hipMalloc(void** p, size_t n) { return allocate(p, n); }
int hipFree(void* p) { return free(p), 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { return allocate(p, n); }
int hipHostFree(void* p) { return free(p), 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, kInvalidValue; }

// ---- streams, events, graphs ----
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = malloc(1), 0; }
int hipStreamDestroy(void* s) { return free(s), 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamIsCapturing(void*, int* st) { return *st = capturing, 0; }
int hipEventCreate(double** e) { return *e = (double*)calloc(1, sizeof(double)), 0; }
int hipEventCreateWithFlags(double** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(double* e) { return free(e), 0; }
int hipEventRecord(double* e, void*) { return *e = now, 0; }
int hipEventSynchronize(double*) { return 0; }
int hipEventElapsedTime(float* ms, double* a, double* b) { return *ms = (float)(*b - *a), 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { return *g = malloc(1), 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { return *x = malloc(1), 0; }
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void* g) { return free(g), 0; }
int hipGraphExecDestroy(void* x) { return free(x), 0; }
}
