// A HIP runtime without a GPU, for tests of the library's host code: device memory is host memory, launches are written down,
// and the kernels that put a plan on the device are carried out, so that a test sees what the device holds.  Loaded
// with RTLD_GLOBAL before the library, whose HIP calls then come here.
#include <cxxabi.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "kernels.h"

using namespace collm;

namespace {

// as in the kernel sources: passes that carry new table addresses, a chunk of a plan as an argument
struct WideArgs : GemmArgs { PlanPatch patch; };
struct SkinnyPassArgs : SkinnyArgs { PlanPatch patch; };
struct MixedPassArgs : GemmArgs { SkinnyPassArgs pass; int mixed_split, mixed_cols; };  // (in the kernels' names: MixedArgs<.., SkinnyPassArgs>)
struct PlanChunk { int32_t v[896]; };

struct Launch {
    std::string name;
    std::vector<unsigned char> first;  // the first argument (of the kernels carried out here)
    uint64_t rest[5];
};

std::map<const void *, std::string> g_names;
std::map<const void *, int> g_lds_attr;
std::set<hipStream_t> g_capturing;
std::vector<Launch> g_graph;
std::string g_log, g_fail;
hipError_t g_error = hipSuccess;
bool g_fail_query = false, g_relaxed = false;
unsigned long long g_capture_id = 0;
const int32_t *g_plan = nullptr;  // where the first upload went: the block of the plan on the device
struct { dim3 grid, block; size_t smem; hipStream_t st; } g_call;

bool has(const std::string &s, const char *part) { return s.find(part) != std::string::npos; }

void copy_patch(const PlanPatch &q)
{
    for (int part = 0; part < kPatchParts; ++part)
        std::memcpy(q.dst + 4 * (size_t)q.lo[part], q.src + 4 * (size_t)q.lo[part], 16 * (size_t)q.n[part]);
    *q.done_host = q.seq;
}

Launch take(const std::string &name, void **args)
{
    Launch l;
    l.name = name;
    size_t bytes = 8;
    int rest = 0;
    if (has(name, "plan_copy_kernel")) rest = 5;
    if (has(name, "plan_words_kernel")) bytes = sizeof(PlanChunk), rest = 2;
    if (has(name, "WideArgs")) bytes = sizeof(WideArgs);
    if (has(name, "SkinnyPassArgs")) bytes = has(name, "MixedArgs") ? sizeof(MixedPassArgs) : sizeof(SkinnyPassArgs);
    l.first.assign((unsigned char *)args[0], (unsigned char *)args[0] + bytes);
    for (int i = 0; i < rest; ++i) {
        l.rest[i] = 0;
        const bool word = (has(name, "plan_copy_kernel") && (i == 1 || i == 4)) || (has(name, "plan_words_kernel") && i == 1);
        std::memcpy(&l.rest[i], args[1 + i], word ? 4 : 8);
    }
    return l;
}

void carry_out(const Launch &l)
{
    const unsigned char *a = l.first.data();
    if (has(l.name, "plan_copy_kernel")) {
        const void *src;
        std::memcpy(&src, a, 8);
        std::memcpy((void *)l.rest[0], src, 16 * (size_t)l.rest[1]);
        *(uint32_t *)l.rest[3] = (uint32_t)l.rest[4];
    } else if (has(l.name, "plan_words_kernel")) {
        std::memcpy((void *)l.rest[0], a, 4 * (size_t)l.rest[1]);
    } else if (has(l.name, "WideArgs")) {
        copy_patch(reinterpret_cast<const WideArgs *>(a)->patch);
    } else if (has(l.name, "MixedArgs") && has(l.name, "SkinnyPassArgs")) {
        copy_patch(reinterpret_cast<const MixedPassArgs *>(a)->pass.patch);
    } else if (has(l.name, "SkinnyPassArgs")) {
        copy_patch(reinterpret_cast<const SkinnyPassArgs *>(a)->patch);
    }
}

hipError_t launch(const void *f, dim3 grid, void **args, size_t smem, hipStream_t st)
{
    const std::string &name = g_names[f];
    if (!g_fail.empty() && has(name, g_fail.c_str())) {
        g_log += "failed " + name + "\n";
        g_fail.clear();
        return g_error = hipErrorLaunchFailure;
    }
    const int attr = g_lds_attr.count(f) ? g_lds_attr[f] : 0;
    char buf[160];
    std::snprintf(buf, sizeof buf, "\t%u %u %u\t%zu\t%d\n", grid.x, grid.y, grid.z, smem, attr);
    g_log += name + buf;
    const Launch l = take(name, args);
    if (!g_plan && (has(name, "plan_copy_kernel") || has(name, "plan_words_kernel"))) g_plan = (const int32_t *)l.rest[0];
    if (g_capturing.count(st)) g_graph.push_back(l);
    else carry_out(l);
    return hipSuccess;
}

void *zeroed(size_t n)
{
    void *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    std::memset(p, 0, (n + 255) / 256 * 256);
    return p;
}

}  // namespace

extern "C" {

// what the tests use
void fake_capture(void *st, int on)
{
    if (on && g_capturing.empty()) ++g_capture_id;
    on ? (void)g_capturing.insert((hipStream_t)st) : (void)g_capturing.erase((hipStream_t)st);
}
void fake_new_graph() { g_graph.clear(); }
void fake_replay() { for (const Launch &l : g_graph) carry_out(l); }
void fake_fail_launch(const char *part) { g_fail = part; }
void fake_fail_query(int on) { g_fail_query = on; }
void fake_new_plan() { g_plan = nullptr; }
const int32_t *fake_plan() { return g_plan; }
const char *fake_log()
{
    static std::string last;
    last.swap(g_log);
    g_log.clear();
    return last.c_str();
}

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    char *s = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    std::string name = s ? s : device;
    std::free(s);
    const size_t end = name.rfind('(');
    if (end != std::string::npos) name.resize(end);
    g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t smem, hipStream_t st)
{
    g_call = {grid, block, smem, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *smem, hipStream_t *st)
{
    *grid = g_call.grid;
    *block = g_call.block;
    *smem = g_call.smem;
    *st = g_call.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t smem, hipStream_t st) { return launch(f, grid, args, smem, st); }
hipError_t hipExtLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t smem, hipStream_t st, hipEvent_t, hipEvent_t, int)
{
    return launch(f, grid, args, smem, st);
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v)
{
    g_lds_attr[f] = v;
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_error;
    g_error = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "an error"; }
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *s)
{
    if (g_fail_query) return hipErrorStreamCaptureImplicit;
    *s = g_capturing.count(st) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t st, hipStreamCaptureStatus *s, unsigned long long *id)
{
    *id = g_capture_id;
    return hipStreamIsCapturing(st, s);
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode)
{
    const hipStreamCaptureMode old = g_relaxed ? hipStreamCaptureModeRelaxed : hipStreamCaptureModeGlobal;
    g_relaxed = *mode == hipStreamCaptureModeRelaxed;
    *mode = old;
    return hipSuccess;
}
hipError_t allocate(void **p, size_t n)
{
    if (!g_capturing.empty() && !g_relaxed) return hipErrorStreamCaptureUnsupported;
    return *p = zeroed(n), hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return allocate(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return allocate(p, n); }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *scratch = zeroed((size_t)16 << 20);
    return *p = scratch, hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { return std::memset(p, 0, sizeof *p), hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)zeroed(8), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free(s), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)zeroed(8), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)zeroed(8), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }

}
