// runtime.cpp -- a model of the HIP runtime for CPU tests of the library's host
// code: device memory is host memory (zeroed), kernels do nothing, and streams,
// events and host synchronisation keep vector clocks, so that a test can ask
// whether one launch is ordered after another, which no run on a GPU can show.
// Built with the host part of every library source by tests/test_host_model.py.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

using Clock = std::map<hipStream_t, long>;    // per stream: the last operation known to be done

static void join(Clock& a, const Clock& b)
{
    for (auto& kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}

struct Launch {
    std::string name;
    Clock at;
};

static std::map<hipStream_t, Clock> streams;
static std::map<hipEvent_t, Clock> events;
static Clock host;
static std::vector<Launch> launches;
static std::map<const void*, std::string>& names()    // filled before this file's own objects exist
{
    static std::map<const void*, std::string> m;
    return m;
}
static long next_handle = 0x1000;
static int capturing = 0, in_capture = 0, mallocs = 0;
static int fail_malloc = -1;          // hipMalloc calls left before one that fails
static long long list_flag = 0;       // what an 8-byte copy to the host delivers
static std::string watched;           // model_watch: the kernel, the index of an int argument, its last value
static int watched_arg, watched_value;
static void (*sync_hook)();           // called by the next hipStreamSynchronize
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static hipStream_t cfg_stream;

static Clock& step(hipStream_t s)     // one more operation on s
{
    Clock& c = streams[s];
    join(c, host);
    ++c[s];
    return c;
}

extern "C" {

// ------------------------------------------------------------ for the tests
hipStream_t model_stream() { return (hipStream_t)next_handle++; }
void model_clear() { launches.clear(); }
long model_now(hipStream_t s) { return streams[s][s]; }
// the launches since model_clear() of kernels whose (mangled) name holds `part`
int model_launches(const char* part)
{
    int n = 0;
    for (auto& l : launches) n += l.name.find(part) != std::string::npos;
    return n;
}
// the launches since model_clear() that do not come after operation `at` of stream s; the first one's name
int model_before(hipStream_t s, long at, char* name, int len)
{
    int n = 0;
    for (auto& l : launches)
        if (l.at[s] < at && n++ == 0) {
            std::strncpy(name, l.name.c_str(), len - 1);
            name[len - 1] = 0;
        }
    return n;
}
// the launches that the next operation on s does not come after
int model_not_joined(hipStream_t s)
{
    Clock c = streams[s];
    join(c, host);
    int n = 0;
    for (auto& l : launches)
        for (auto& kv : l.at)
            if (c[kv.first] < kv.second) {
                ++n;
                break;
            }
    return n;
}
void model_watch(const char* part, int arg)
{
    watched = part;
    watched_arg = arg;
}
int model_watched() { return watched_value; }
void model_on_sync(void (*f)()) { sync_hook = f; }
int model_created_in_capture() { return in_capture; }
int model_mallocs() { return mallocs; }
void model_fail_malloc(int after) { fail_malloc = after; }
void model_list_flag(long long v) { list_flag = v; }

// ------------------------------------------------------------------ runtime
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize()
{
    for (auto& kv : streams) join(host, kv.second);
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "model"; }

hipError_t hipMalloc(void** p, size_t n)
{
    if (capturing) ++in_capture;
    ++mallocs;
    if (fail_malloc >= 0 && fail_malloc-- == 0) return hipErrorOutOfMemory;
    *p = std::calloc(n, 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }

hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    step(st);
    std::memcpy(d, s, n);
    if (k == hipMemcpyDeviceToHost && n == sizeof(list_flag)) std::memcpy(d, &list_flag, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t s)
{
    step(s);
    std::memset(p, v, n);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    if (capturing) ++in_capture;
    *s = model_stream();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    join(host, streams[s]);
    if (void (*f)() = sync_hook) {
        sync_hook = nullptr;
        f();
    }
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    join(streams[s], events[e]);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    if (capturing) ++in_capture;
    *e = (hipEvent_t)next_handle++;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { events.erase(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    events[e] = streams[s];
    join(events[e], host);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { join(host, events[e]); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }

// a captured stream's work counts as done where it is captured
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { ++capturing; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { --capturing; *g = (hipGraph_t)next_handle++; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = (hipGraphExec_t)next_handle++;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { step(s); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

// ----------------------------------------------------------------- launches
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    cfg_grid = g;
    cfg_block = b;
    cfg_shared = sh;
    cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *sh = cfg_shared;
    *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s)
{
    if (!watched.empty() && names()[f].find(watched) != std::string::npos)
        watched_value = *static_cast<int*>(args[watched_arg]);
    launches.push_back(Launch{names()[f], step(s)});
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
