// The HIP runtime calls that libpfb.so makes, on the host and without a
// device: memory is host memory, launches and synchronisations are recorded,
// and one kernel can be made to fail to launch. The streaming copies, whose
// effect a test looks at, are carried out. Loaded ahead of the real runtime.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> names;
std::string events, failing, slow;
int cus = 256;
size_t allocated = 0;
float clock_ms = 0.0f, slow_ms = 1.0f;
hipError_t last = hipSuccess;
struct Call {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} call;
char symbol[64 << 20];

void record(const std::string &what) { events += what + "\n"; }

template <class T> T arg(void **args, int i) { return *static_cast<T *>(args[i]); }

// copy_blocks_kernel and rotate_history_kernel (csrc/stream.hip)
void copy_blocks(void **args)
{
    const char *src = arg<const char *>(args, 0);
    const int64_t sstr = arg<int64_t>(args, 1), dstr = arg<int64_t>(args, 3), bytes = arg<int64_t>(args, 4);
    char *dst = arg<char *>(args, 2);
    for (int64_t b = 0; b < arg<int64_t>(args, 5); ++b)
        src ? (void)std::memmove(dst + b * dstr, src + b * sstr, bytes) : (void)std::memset(dst + b * dstr, 0, bytes);
}
void rotate_history(void **args, int64_t unit)
{
    char *hist = arg<char *>(args, 0), *xb = arg<char *>(args, 1);
    const int64_t stride = arg<int64_t>(args, 2), tail = arg<int64_t>(args, 3), bytes = arg<int64_t>(args, 4) * unit;
    for (int64_t b = 0; b < arg<int64_t>(args, 5); ++b) {
        std::memcpy(xb + b * stride, hist + b * bytes, bytes);
        std::memcpy(hist + b * bytes, xb + b * stride + tail, bytes);
    }
}
} // namespace

extern "C" {

// the test's side
void host_cus(int n) { cus = n; }
void host_fail(const char *kernel) { failing = kernel; }                          // "" none
void host_time(const char *kernel, float ms) { slow = kernel, slow_ms = ms; }     // others take 1 ms
size_t host_allocated() { return allocated; }
const char *host_events()
{
    static std::string out;
    out.swap(events);
    events.clear();
    return out.c_str();
}

// registration and launch
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) { call = {g, b, s, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st)
{
    *g = call.grid, *b = call.block, *s = call.shared, *st = call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t)
{
    const std::string &n = names[f];
    if (!failing.empty() && n.find(failing) != std::string::npos)
        return last = hipErrorLaunchFailure;
    record("launch " + n + " " + std::to_string((long long)g.x * g.y * g.z) + " " + std::to_string(b.x));
    clock_ms += !slow.empty() && n.find(slow) != std::string::npos ? slow_ms : 1.0f;
    if (n.find("copy_blocks_kernel") != std::string::npos)
        copy_blocks(args);
    else if (n.find("rotate_history_kernel") != std::string::npos)
        rotate_history(args, n.find("HIP_vector_type") != std::string::npos ? 16 : 1);
    return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t) { return "host"; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return hipSuccess; }

// device and memory
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = cus; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = cus;
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    allocated += n;
    return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    record("copy " + std::to_string(n));
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = symbol; return hipSuccess; }

// events and graphs
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(new float(0.0f)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<float *>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *reinterpret_cast<float *>(e) = clock_ms; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { record("wait"); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    *ms = *reinterpret_cast<float *>(b) - *reinterpret_cast<float *>(a);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { record("wait"); return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t *g, unsigned) { *g = reinterpret_cast<hipGraph_t>(1); return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t *n, hipGraph_t, const hipGraphNode_t *, size_t, const hipKernelNodeParams *)
{
    *n = reinterpret_cast<hipGraphNode_t>(1);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(1);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { record("graph"); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

} // extern "C"
