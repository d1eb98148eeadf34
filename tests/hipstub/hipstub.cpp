// A HIP runtime for the CPU, for tests of libsmx's host side: loaded (globally) before
// libsmx.so, it takes the place of the runtime's functions that the library calls.
// Device memory is host memory, zero where it is fresh; kernels do not run, they are
// written to a log (name and grid).  Of their effects only those that the host's
// control flow reads are played, in stream order and as late as a device might: when
// the host asks for the stream's progress or waits.  They are the cleared
// finished-group counter, the progress word of a square and the counter once the
// update of step `finish` is through.
#include <cxxabi.h>

#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <string>

#include "smx.h"
#include "smx_internal.h"

namespace {

std::map<const void *, std::string> names;
std::deque<std::function<void()>> pending;
std::string log_text;
int finish = 1 << 30, fail_event = -1, events = 0;

void drain()
{
    while (!pending.empty()) {
        pending.front()();
        pending.pop_front();
    }
}

// The n-th integer of "kernel<a, b, ...>".
int targ(const std::string &s, int n)
{
    size_t p = s.find('<');
    while (n-- > 0 && p != std::string::npos) p = s.find(',', p + 1);
    return p == std::string::npos ? -1 : std::atoi(s.c_str() + p + 1);
}

hipError_t new_event(hipEvent_t *e)
{
    if (events++ == fail_event) return hipErrorOutOfMemory;
    *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
    return hipSuccess;
}

}  // namespace

extern "C" {

// ---- for the tests ----
void stub_set(int finish_step, int fail_event_at)
{
    finish = finish_step;
    fail_event = fail_event_at;
    events = 0;
}
int stub_events() { return events; }                    // created since stub_set
const char *stub_log() { return log_text.c_str(); }
void stub_clear_log() { log_text.clear(); }

// ---- kernels ----
void **__hipRegisterFatBinary(const void *) { return static_cast<void **>(std::malloc(8)); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = st == 0 ? d : name;
    std::free(d);
    // "void smx::(anonymous namespace)::kernel<...>(...)" -> "kernel<...>"
    const size_t tail = s.rfind("namespace)::");
    if (tail != std::string::npos) s = s.substr(tail + 12);
    s = s.substr(0, s.find('('));
    const size_t at = s.rfind("::", s.find('<'));
    names[host] = at == std::string::npos ? s : s.substr(at + 2);
}
static dim3 cfg_grid, cfg_block;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    cfg_grid = grid;
    cfg_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *st)
{
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = 0;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t)
{
    const std::string &n = names[f];
    log_text += n + " " + std::to_string(grid.x) + "\n";
    const std::string base = n.substr(0, n.find('<'));
    if (base == "clear_state_kernel") {
        int32_t *nd = *static_cast<int32_t **>(args[8]);
        if (nd) pending.push_back([=] { *nd = 0; });
        return hipSuccess;
    }
    int mode = -1, at = 5;
    if (base == "ns_f64_kernel" || base == "ns_f32_kernel") mode = targ(n, 0);
    else if (base == "ns_words_kernel" || base == "ns_words32_kernel" || base == "ns_words256_kernel") mode = targ(n, 2);
    else if (base == "ns_words_persistent") mode = targ(n, 2), at = 7;
    if (mode < 0) return hipSuccess;
    const smx::IterState it = *static_cast<smx::IterState *>(args[at]);
    const int k = *static_cast<int *>(args[at + 1]), last = finish;
    const bool square = mode == 0 || mode == 5 || (mode == 2 && base != "ns_f64_kernel");
    pending.push_back([=] {
        if (square && it.poll) *it.poll = (unsigned long long)(it.poll_tag + (uint32_t)k) << 32 | (unsigned)*it.ndone;
        if (mode == 1 && k >= last) *it.ndone = 1 << 20;
    });
    return hipSuccess;
}

// ---- memory ----
hipError_t hipMalloc(void **p, size_t n) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { drain(); std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { drain(); std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { drain(); std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemGetInfo(size_t *fr, size_t *tot) { *fr = *tot = 288ull << 30; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *scratch = std::calloc(1, (size_t)SMX_STATIC_SCRATCH_BYTES + ((size_t)64 << 20));
    *p = scratch;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }

// ---- device, streams, events ----
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    std::strcpy(p->gcnArchName, "stub");
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 3; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t *s) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return hipStreamCreate(s); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { drain(); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t)
{
    if (pending.empty()) return hipSuccess;
    pending.front()();
    pending.pop_front();
    return hipErrorNotReady;
}
hipError_t hipEventCreate(hipEvent_t *e) { return new_event(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return new_event(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(reinterpret_cast<void *>(e)); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { drain(); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }

}  // extern "C"
