// Stand-ins for the HIP runtime calls that libfdbb.so makes, for tests of its
// host code without a device.  Loaded with global symbols before the library,
// they take the place of the runtime's: device memory is host memory, copies
// happen at once, kernels do not run.  Each launch is logged with its kernel,
// shape and dynamic LDS; captures record launches and copies, and a graph
// launch runs them.  Calls can be made to fail by name.
#ifndef __HIP_PLATFORM_AMD__
#define __HIP_PLATFORM_AMD__
#endif
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string kernel;
    int grid, block;
    int64_t lds;
    int64_t units;  // of a batch launch: the second word of its header, when it runs
    bool replay;
};

std::map<const void *, std::string> g_names;
std::vector<Launch> g_log;
std::string g_text;
std::set<std::string> g_failing;
std::map<hipStream_t, std::vector<std::function<void(bool)>>> g_captures;
uintptr_t g_next = 0x1000;

hipError_t failing(const char *call) { return g_failing.count(call) ? hipErrorInvalidValue : hipSuccess; }

// Runs `op` now, or records it where the stream is being captured.
void on(hipStream_t s, std::function<void(bool)> op)
{
    auto it = g_captures.find(s);
    if (it == g_captures.end()) op(false);
    else it->second.push_back(op);
}

}  // namespace

extern "C" {

const char *host_log()
{
    g_text.clear();
    for (const Launch &l : g_log)
        g_text += l.kernel + " " + std::to_string(l.grid) + " " + std::to_string(l.block) + " " +
                  std::to_string(l.lds) + " " + std::to_string(l.units) + " " + (l.replay ? "1" : "0") + "\n";
    g_log.clear();
    return g_text.c_str();
}

void host_fail(const char *call, int on)
{
    if (on) g_failing.insert(call);
    else g_failing.erase(call);
}

void **__hipRegisterFatBinary(const void *) { return new void *(nullptr); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

hipError_t hipGetDevice(int *dev)
{
    *dev = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    if (hipError_t e = failing("hipMemcpyAsync")) return e;
    on(st, [=](bool) { std::memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t)++g_next;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return failing("hipEventRecord"); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = (hipStream_t)++g_next;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    if (failing("hipStreamIsCapturing")) return hipErrorStreamCaptureImplicit;
    *st = g_captures.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    g_captures[s].clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    *g = (hipGraph_t) new std::vector<std::function<void(bool)>>(g_captures[s]);
    g_captures.erase(s);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *x = (hipGraphExec_t) new std::vector<std::function<void(bool)>>(*(std::vector<std::function<void(bool)>> *)g);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete (std::vector<std::function<void(bool)>> *)g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete (std::vector<std::function<void(bool)>> *)x;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s)
{
    // on a stream that is being captured too, as the runtime does
    (void)s;
    for (const auto &op : *(std::vector<std::function<void(bool)>> *)x) op(true);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *, const void *) { return hipErrorInvalidValue; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *table = std::calloc(1, 1 << 20);
    *p = table;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t s)
{
    if (hipError_t e = failing("hipLaunchKernel")) return e;
    const std::string name = g_names[fn];
    const int64_t *header = name.find("k_batch") == std::string::npos ? nullptr : *(const int64_t **)args[2];
    on(s, [=](bool replay) {
        g_log.push_back({name, (int)grid.x, (int)block.x, (int64_t)lds, header ? header[1] : 0, replay});
    });
    return hipSuccess;
}

}  // extern "C"
