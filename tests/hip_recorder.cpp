// A stand-in for the HIP runtime that runs on the CPU: device memory is host
// memory, kernels are not run but recorded.  Loaded ahead of the library
// (RTLD_GLOBAL), so that the launches an entry point makes can be checked
// without a GPU (test_dispatch.py).
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;
    dim3 grid, block;
    const void* arg[2]; // the first two parameters
    int rev;            // step kernels: Geom::rev
};
std::map<const void*, std::string>& names()
{
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<Launch> launches;
std::map<void*, size_t> blocks; // live device memory
int64_t live = 0, peak = 0;
int capturing = 0;
dim3 next_grid, next_block;
size_t next_lds = 0;
hipStream_t next_stream = nullptr;
char symbol_memory[1 << 21];

hipError_t take(void** p, size_t n)
{
    *p = std::calloc(n ? n : 1, 1);
    if (!*p) return hipErrorOutOfMemory;
    blocks[*p] = n;
    live += (int64_t)n;
    if (live > peak) peak = live;
    return hipSuccess;
}

} // namespace

extern "C" {

// what the tests read
int rec_count() { return (int)launches.size(); }
const char* rec_name(int i) { return launches[i].name.c_str(); }
const void* rec_arg(int i, int k) { return launches[i].arg[k]; }
int64_t rec_threads(int i)
{
    const Launch& l = launches[i];
    return (int64_t)l.grid.x * l.grid.y * l.grid.z * l.block.x * l.block.y * l.block.z;
}
int rec_rev(int i) { return launches[i].rev; }
void rec_clear() { launches.clear(); }
int64_t rec_live_bytes() { return live; }
int64_t rec_peak_bytes() { return peak; }
void rec_set_capturing(int on) { capturing = on; }

// registration and launches
void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* name, const char*, unsigned, void*, void*, dim3*, dim3*, int*)
{
    names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st)
{
    next_grid = g;
    next_block = b;
    next_lds = lds;
    next_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st)
{
    *g = next_grid;
    *b = next_block;
    *lds = next_lds;
    *st = next_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t)
{
    Launch l{names()[f], g, b, {nullptr, nullptr}, 0};
    for (int k = 0; k < 2; ++k) std::memcpy(&l.arg[k], args[k], sizeof(void*));
    const auto is = [&](const char* part) { return l.name.find(part) != std::string::npos; };
    const int geom = is("k_mhd_step") ? 4 : is("k_step_aa") ? 1 : is("k_step_ab") || is("k_step_mlp") ? 2 : -1;
    if (geom >= 0) l.rev = static_cast<const int*>(args[geom])[5]; // nx, ny, nz, nxy, N, rev
    launches.push_back(l);
    return hipSuccess;
}

// memory
hipError_t hipMalloc(void** p, size_t n) { return take(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = std::calloc(n ? n : 1, 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p)
{
    auto it = blocks.find(p);
    if (it != blocks.end()) {
        live -= (int64_t)it->second;
        blocks.erase(it);
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n)
{
    if (v || n < (1 << 20)) std::memset(d, v, n); // large buffers are cleared once, when they are new and zero
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t)
{
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = symbol_memory;
    return hipSuccess;
}

// device, streams, events, graphs
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256
         : a == hipDeviceAttributeMaxSharedMemoryPerMultiprocessor ? 163840 : 0;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int)
{
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t)symbol_memory;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)symbol_memory;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = (hipGraphExec_t)symbol_memory;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)symbol_memory;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}

} // extern "C"
