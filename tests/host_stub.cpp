// host_stub.cpp -- a HIP runtime that launches nothing, for CPU tests of the
// library's host code (planning, workspaces, the sequence of launches): every
// kernel launch is recorded by its kernel's name, memory is reserved address
// space that nobody touches, and an allocation above a limit or a launch of a
// chosen kernel can be made to fail.  Linked in place of the HIP runtime.
#include <hip/hip_runtime.h>

#include <cxxabi.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& kernels()
{
    static std::map<const void*, std::string> m;
    return m;
}
std::map<void*, size_t> g_blocks;
std::string g_log;
std::string g_bad_kernel;
size_t g_alloc_limit = ~(size_t)0;
size_t g_largest = 0;
long g_bad_skip = 0;
hipError_t g_error = hipSuccess;

struct Dims {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
} g_dims;
}  // namespace

extern "C" {

// ---- control: the log of kernel names since the last call, one a line
const char* stub_log()
{
    static std::string out;
    out.swap(g_log);
    g_log.clear();
    return out.c_str();
}
void stub_alloc_limit(size_t bytes) { g_alloc_limit = bytes; }
// launches of kernels whose name contains `name` fail, after `skip` of them
void stub_fail_kernel(const char* name, long skip)
{
    g_bad_kernel = name;
    g_bad_skip = skip;
}
// bytes of the largest allocation since the last call
size_t stub_largest()
{
    const size_t b = g_largest;
    g_largest = 0;
    return b;
}
// bytes allocated now
size_t stub_total()
{
    size_t b = 0;
    for (const auto& kv : g_blocks) b += kv.second;
    return b;
}

// ---- runtime
void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*)
{
    int status = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    kernels()[host] = d ? d : name;
    std::free(d);
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream)
{
    g_dims = { grid, block, shmem, stream };
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream)
{
    *grid = g_dims.grid;
    *block = g_dims.block;
    *shmem = g_dims.shmem;
    *stream = g_dims.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t)
{
    const std::string& name = kernels()[f];
    if (!g_bad_kernel.empty() && name.find(g_bad_kernel) != std::string::npos && g_bad_skip-- <= 0)
        return g_error = hipErrorLaunchFailure;
    g_log += name + "\n";
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes)
{
    if (bytes > g_largest) g_largest = bytes;
    if (bytes > g_alloc_limit) return g_error = hipErrorOutOfMemory;
    void* m = mmap(nullptr, bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return g_error = hipErrorOutOfMemory;
    g_blocks[m] = bytes;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (g_blocks.count(p)) munmap(p, g_blocks[p]);
    g_blocks.erase(p);
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = g_error;
    g_error = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static char symbol[1 << 20];
    *p = symbol;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void*, size_t bytes, hipMemcpyKind kind, hipStream_t)
{
    if (kind == hipMemcpyDeviceToHost) std::memset(dst, 0, bytes);
    g_log += "copy\n";
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t bytes, hipMemcpyKind kind)
{
    return hipMemcpyAsync(dst, src, bytes, kind, nullptr);
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* prop, int)
{
    std::memset(prop, 0, sizeof *prop);
    prop->multiProcessorCount = 256;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)&g_dims;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    static float t = 0.0f;
    *ms = t += 1.0f;   // later is slower
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t)&g_dims;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)&g_dims;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = (hipGraphExec_t)&g_dims;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t)
{
    g_log += "graph\n";
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
