// fake_hip.cpp - a HIP runtime of the host, for tests of the library's host code
// without a GPU. Device memory is host memory; kernels do nothing but ssa_upload, which
// copies as the real one does. Calls are written to a log, one line each. What a
// test sets: occupancies, the capture status of streams, the event that fails.
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <sstream>
#include <string>

namespace {
std::ostringstream g_log;
std::map<std::string, long> g_set;
std::string g_text;
long g_events = 0;
void *g_tables = nullptr;   // where the last copy or first upload since it was taken went

long setting(const char *name, long otherwise)
{
    auto it = g_set.find(name);
    return it == g_set.end() ? otherwise : it->second;
}

const char *name_of(hipFunction_t f) { return (const char *)f; }
}  // namespace

extern "C" {

void fake_set(const char *name, long v) { g_set[name] = v; }

void fake_reset()
{
    g_set.clear();
    g_log.str("");
    g_events = 0;
}

const char *fake_log()
{
    g_text = g_log.str();
    return g_text.c_str();
}

void *fake_tables()
{
    void *p = g_tables;
    return g_tables = nullptr, p;
}

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipModuleLoadData(hipModule_t *m, const void *) { return *m = (hipModule_t)1, hipSuccess; }

hipError_t hipModuleGetFunction(hipFunction_t *f, hipModule_t, const char *name)
{
    return *f = (hipFunction_t)strdup(name), hipSuccess;
}

hipError_t hipFuncGetAttribute(int *v, hipFunction_attribute, hipFunction_t f)
{
    // static LDS of the pipelined kernels, none where their ring does not fit
    const std::string n = name_of(f);
    *v = n == "ssa_kernel_pl" ? (int)setting("pl_lds", 4096) : n == "ssa_kernel_ph" ? (int)setting("ph_lds", 4096) : 0;
    return hipSuccess;
}

hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = (int)setting("cus", 256), hipSuccess; }

hipError_t hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(int *n, hipFunction_t f, int block, size_t)
{
    const std::string name = name_of(f);
    *n = name == "ssa_kernel" ? (int)setting("waves_per_cu", 8) * 64 / block : name == "ssa_kernel_ph" ? 2 : 1;
    return hipSuccess;
}

hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned gx, unsigned, unsigned, unsigned bx, unsigned, unsigned,
                                 unsigned lds, hipStream_t, void **args, void **)
{
    const std::string name = name_of(f);
    g_log << "launch " << name << " " << gx << " " << bx << " " << lds << "\n";
    if (name == "ssa_upload") {
        if (!g_tables)
            g_tables = *(void **)args[0];
        std::memcpy(*(void **)args[0], args[2], 4 * (size_t) * (unsigned *)args[1]);
    }
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    g_log << "malloc " << n << "\n";
    return *p = std::calloc(1, n), hipSuccess;
}

hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }

hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    g_log << "memcpy " << n << "\n";
    return std::memcpy(d, s, n), hipSuccess;
}

hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    g_log << "memcpy_async " << n << "\n";
    if (!setting("capturing", 0)) {   // (a captured copy happens when the graph is launched)
        g_tables = d;
        std::memcpy(d, s, n);
    }
    return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t *e)
{
    if (++g_events == setting("fail_event", -1))
        return *e = nullptr, hipErrorOutOfMemory;
    return *e = (hipEvent_t)std::malloc(1), hipSuccess;
}

hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }

hipError_t hipEventSynchronize(hipEvent_t)
{
    g_log << "event_synchronize\n";
    return hipSuccess;
}

hipError_t hipGetSymbolAddress(void **p, const void *s) { return *p = const_cast<void *>(s), hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }

hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    return *s = setting("capturing", 0) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone, hipSuccess;
}

hipError_t hipStreamSynchronize(hipStream_t)
{
    g_log << "stream_synchronize\n";
    return hipSuccess;
}

hiprtcResult hiprtcCreateProgram(hiprtcProgram *, const char *, const char *, int, const char *const *,
                                 const char *const *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcCompileProgram(hiprtcProgram, int, const char *const *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcGetProgramLogSize(hiprtcProgram, size_t *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcGetProgramLog(hiprtcProgram, char *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcGetCodeSize(hiprtcProgram, size_t *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcGetCode(hiprtcProgram, char *) { return HIPRTC_ERROR_INTERNAL_ERROR; }
hiprtcResult hiprtcDestroyProgram(hiprtcProgram *) { return HIPRTC_SUCCESS; }

}  // extern "C"
