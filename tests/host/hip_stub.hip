// hip_stub.hip - a stand-in for the HIP runtime, for tests of the library's host code on a machine
// without a GPU (test support; built with hipcc for the host only, loaded before libhjw.so so
// that the library's calls bind to it).
//
// Device memory is host memory, tagged with the device it was allocated on.  Launches are
// written to a log, and the kernels that move a grid's step record are played: a step adds
// g_dt to t.  What a resident launch does is chosen by the test: it steps, it gives its meeting
// up, or it stops answering.  phi itself is never computed.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "hjw_resident.h"
#include "hjw_tile.h"

using namespace hjw;

namespace {

int g_device = 0, g_devices = 2, g_cus = 256, g_per_cu = 4;
// What each resident launch does: '0' steps, '1' gives its meeting up, '2' stops answering at its
// second step; the last one for all that follow.
std::string g_modes = "0";
double g_dt = 1.0 / 1024;
void (*g_hook)() = nullptr;    // called at each resident launch, before it plays
std::string g_log;
std::map<const void*, std::string> g_names;
std::map<const void*, size_t> g_vars;              // device variables' sizes
std::map<char*, std::pair<size_t, int>> g_memory;   // base -> bytes, device
std::map<void*, int> g_streams;

struct Captured {
    std::string name;
    std::vector<char> args;
    dim3 grid, block;
};
bool g_capturing = false;
std::vector<Captured> g_capture;
std::vector<std::vector<Captured>*> g_graphs;

void note(const char* fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_log += buf;
    g_log += '\n';
}
int device_of(const void* p) {
    for (const auto& m : g_memory)
        if (p >= m.first && p < m.first + m.second.first) return m.second.second;
    return -1;
}
bool open(const DevState& s) { return !s.bad && s.t < s.t_final && s.steps_left > 0; }
void advance(DevState& s) {
    s.dt = g_dt < s.t_final - s.t ? g_dt : s.t_final - s.t;
    s.t = g_dt < s.t_final - s.t ? s.t + g_dt : s.t_final;
    s.steps += 1;
    s.steps_left -= 1;
}
template <typename T, typename P>
void play_stage(const void* arg) {
    const auto& a = *static_cast<const StageArgs<T, P>*>(arg);
    DevState s = a.st[a.par];
    s.active = open(s) ? 1 : 0;
    if (s.active) advance(s);
    a.st[a.par ^ 1] = s;
}
// The bytes of a kernel's first argument, where the kernel is played later from a graph.
size_t arg_bytes(const std::string& n) {
    return n.find("Idd") != n.npos   ? sizeof(StageArgs<double, double>)
           : n.find("Ifd") != n.npos ? sizeof(StageArgs<float, double>)
                                     : sizeof(StageArgs<float, float>);
}
template <typename T, typename P>
int parity(const void* arg) {
    return static_cast<const StageArgs<T, P>*>(arg)->par;
}
void play(const std::string& n, const void* arg0, void** args, dim3 grid, dim3 block) {
    const auto is = [&](const char* k) { return n.find(k) != n.npos; };
    const auto arg = [&](int k) { return args[k]; };
    if (is("k_resident_begin")) {
        DevState* st = *static_cast<DevState**>(arg(0));
        ResidentCtl* ctl = *static_cast<ResidentCtl**>(arg(1));
        if (*static_cast<int*>(arg(6)) && st->pad[0] != 1) {
            ctl->go = 2;
            return;
        }
        *ctl = ResidentCtl{};
        st->pad[0] = 0;
        if (*static_cast<int*>(arg(2))) {
            st->t_final = *static_cast<double*>(arg(3));
            st->cfl = *static_cast<double*>(arg(4));
            st->steps_left = *static_cast<int64_t*>(arg(5));
        }
    } else if (is("k_resident")) {
        const ResidentArgs& r = *static_cast<const ResidentArgs*>(arg(1));
        note("resident count=%d block=%u epoch=%u steps=%d mail_device=%d", r.count, block.x, r.epoch,
             r.max_steps, device_of(r.flux_mail));
        if (r.ctl->go) return;
        if (g_hook) g_hook();
        const char mode = g_modes[0];
        if (g_modes.size() > 1) g_modes.erase(0, 1);
        if (mode == '1') return;
        const int par = is("Idd")   ? parity<double, double>(arg0)
                        : is("Ifd") ? parity<float, double>(arg0)
                                    : parity<float, float>(arg0);
        DevState& s = r.state[par];
        for (int k = 0; k < r.max_steps && open(s); ++k) {
            if (mode == '2' && k == 1) {
                s.pad[0] = 2;
                return;
            }
            advance(s);
        }
        s.pad[0] = 1;
    } else if (is("k_stage") && is("Li0E")) {   // a step's first stage
        note("step grid=%u block=%u%s", grid.x, block.x, is("Lb0ELb1E") ? " dense" : "");
        if (is("Idd")) play_stage<double, double>(arg0);
        else if (is("Ifd")) play_stage<float, double>(arg0);
        else play_stage<float, float>(arg0);
    } else if (is("k_set_target")) {
        DevState* st = *static_cast<DevState**>(arg(0));
        st->t_final = *static_cast<double*>(arg(1));
        st->cfl = *static_cast<double*>(arg(2));
        st->steps_left = *static_cast<int64_t*>(arg(3));
    } else if (is("k_reset")) {
        DevState* st = *static_cast<DevState**>(arg(0));
        st[0] = st[1] = DevState{};
    } else if (is("k_clear_words")) {
        note("clear device=%d", device_of(*static_cast<void**>(arg(0))));
    }
}
}  // namespace

extern "C" {

// ------------------------------------------------------------------ for the test
void stub_setup(int devices, int cus, int per_cu) {
    g_devices = devices;
    g_cus = cus;
    g_per_cu = per_cu;
}
void stub_modes(const char* modes) { g_modes = modes; }
void stub_hook(void (*f)()) { g_hook = f; }
size_t stub_variables() {
    size_t sum = 0;
    for (const auto& v : g_vars) sum += v.second;
    return sum;
}
const char* stub_log() { return g_log.c_str(); }
void stub_clear_log() { g_log.clear(); }
void* stub_malloc(size_t bytes, int device) {
    char* p = static_cast<char*>(aligned_alloc(256, (bytes + 255) / 256 * 256));
    memset(p, 0, bytes);
    g_memory[p] = {bytes, device};
    return p;
}

// ------------------------------------------------------------------ the runtime's functions
void** __hipRegisterFatBinary(const void*) {
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned int, void*,
                           void*, void*, void*, int*) {
    g_names[host] = name;
}
void __hipRegisterVar(void**, void* host, char*, char*, int, size_t bytes, int, int) {
    g_vars[host] = bytes;
}

struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
static thread_local Config g_config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    g_config = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *shared = g_config.shared;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    const std::string& n = g_names[f];
    if (g_capturing) {
        const char* a = static_cast<const char*>(args[0]);
        g_capture.push_back({n, std::vector<char>(a, a + arg_bytes(n)), grid, block});
    } else {
        play(n, args[0], args, grid, block);
    }
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) {
    if (d < 0 || d >= g_devices) return hipErrorInvalidDevice;
    g_device = d;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? g_cus : 100000;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = g_per_cu;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    *p = stub_malloc(n, g_device);
    note("malloc device=%d", g_device);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    note("free device=%d", device_of(p));
    g_memory.erase(static_cast<char*>(p));
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* host) {
    *p = stub_malloc(g_vars[host], g_device);
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) {
    *s = reinterpret_cast<hipStream_t>(new int(0));
    g_streams[*s] = g_device;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
    const auto it = g_streams.find(s);
    *d = it == g_streams.end() ? g_device : it->second;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { g_streams.erase(s); delete reinterpret_cast<int*>(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    g_capturing = true;
    g_capture.clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    g_capturing = false;
    g_graphs.push_back(new std::vector<Captured>(g_capture));
    *g = reinterpret_cast<hipGraph_t>(g_graphs.back());
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    *x = reinterpret_cast<hipGraphExec_t>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    note("graph");
    for (auto& c : *reinterpret_cast<std::vector<Captured>*>(x))
        play(c.name, c.args.data(), nullptr, c.grid, c.block);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.0f; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

}  // extern "C"
