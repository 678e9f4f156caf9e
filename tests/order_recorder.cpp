// The HIP runtime and the kernel launches that phx_api.cpp calls, replaced by a record of their
// order, so that the host code's waits between streams can be checked without a GPU.
//
// Every launch, upload and synchronous copy is an operation with a number, which reads and writes
// the context's workspace, its parameter block or its tables.  A stream knows the operations that are
// complete when its next one starts: its own, those of the events that it waited for, and those that
// the host had waited for when it issued the operation.  An operation that starts without knowing an
// earlier one with which it may not overlap is written down.  (The workspace of phx_trace_noalloc is not
// a context's: the caller serialises those calls.)
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../paper_1504_06570_amd/csrc/phx_internal.h"

namespace {

typedef std::set<int> Known;
std::map<void*, Known> g_stream, g_event;
std::map<void*, bool> g_capturing;
Known g_host;
struct Op {
    std::string name;
    unsigned reads, writes;
};
std::vector<Op> g_ops;
enum : unsigned { kWork = 1, kParams = 2, kTables = 4 };
std::string g_overlaps;
int g_resources, g_capture_events;   // allocations, frees, streams, events; event calls while capturing
int g_handles;

void join(Known& a, const Known& b) { a.insert(b.begin(), b.end()); }

std::string label(int i) { return g_ops[(size_t)i].name + "#" + std::to_string(i); }

void check(const Known& k) {
    const int id = (int)g_ops.size() - 1;
    const Op& o = g_ops.back();
    for (int j = 0; j < id; ++j) {
        const Op& p = g_ops[(size_t)j];
        if (!((o.writes & (p.reads | p.writes)) | (o.reads & p.writes))) continue;
        if (!k.count(j)) g_overlaps += label(id) + " may overlap " + label(j) + "\n";
    }
}

hipError_t on_stream(const char* name, hipStream_t s, unsigned reads = kParams | kTables,
                     unsigned writes = kWork) {
    if (g_capturing[s]) return hipSuccess;   // runs when its graph does
    g_ops.push_back({name, reads, writes});
    Known& k = g_stream[s];
    join(k, g_host);
    check(k);
    k.insert((int)g_ops.size() - 1);
    return hipSuccess;
}

hipError_t on_host(const char* name) {   // complete when the call returns
    g_ops.push_back({name, 0, kTables});
    check(g_host);
    g_host.insert((int)g_ops.size() - 1);
    return hipSuccess;
}

void host_waits_for_all() {
    for (int i = 0; i < (int)g_ops.size(); ++i) g_host.insert(i);
}

template <class T>
hipError_t handle(T* out) {
    ++g_resources;
    *out = (T)(uintptr_t)(0x1000 + 16 * ++g_handles);
    return hipSuccess;
}

}  // namespace

extern "C" {

void rec_reset() {
    g_stream.clear();
    g_event.clear();
    g_host.clear();
    g_ops.clear();
    g_overlaps.clear();
    g_resources = g_capture_events = 0;
}
const char* rec_overlaps() { return g_overlaps.c_str(); }
int rec_operations() { return (int)g_ops.size(); }
int rec_resources() { return g_resources; }
int rec_capture_events() { return g_capture_events; }
void rec_capture(void* stream, int on) { g_capturing[stream] = on != 0; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {   // the header's versioned name
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { ++g_resources; *p = std::calloc(n ? n : 1, 1); return hipSuccess; }
hipError_t hipFree(void* p) {   // waits for the device
    if (p) {
        ++g_resources;
        host_waits_for_all();
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return on_host("copy");
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    return on_stream("upload", st, 0, kParams);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
    std::memset(d, v, n);
    return on_stream("fill", st, 0, kTables);
}
hipError_t hipDeviceSynchronize() { host_waits_for_all(); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { join(g_host, g_stream[s]); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { join(g_host, g_event[e]); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return handle(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return handle(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    g_capture_events += g_capturing[s];
    Known k = g_stream[s];
    join(k, g_host);
    g_event[e] = k;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    g_capture_events += g_capturing[s];
    join(g_stream[s], g_event[e]);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return handle(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = g_capturing[s] ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    g_capturing[s] = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { g_capturing[s] = false; return handle(g); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    return handle(x);
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return on_stream("graph", s); }

}  // extern "C"

namespace phx {
hipError_t scratch_address(int, void** out) {
    static std::vector<unsigned char> a(kScratchBytes);
    *out = a.data();
    return hipSuccess;
}
hipError_t launch_prefix(const DevSource*, int, int, uint64_t*, int32_t*, uint64_t, uint32_t,
                         hipStream_t s) {
    return on_stream("prefix", s, kTables, 0);
}
hipError_t launch_trace(const DevParams*, const Launch&, const Workspace& W, int, const LaunchConfig&,
                        hipStream_t s, const Pipe&, const Timing&) {
    if (W.buffers == 1) return on_stream("trace_noalloc", s, kParams | kTables, 0);
    return on_stream("trace", s);
}
hipError_t launch_adjoint(const DevParams*, const Launch&, const Workspace&, int,
                          const LaunchConfig&, const Adjoint&, double*, double*, hipStream_t s,
                          const Pipe&, const Timing&) {
    return on_stream("adjoint", s);
}
hipError_t launch_readout(const ReadoutJob&, hipStream_t s) { return on_stream("readout", s, 0); }
hipError_t launch_moments(const unsigned long long*, int, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_seeds(const unsigned long long*, int, const double*, double*, hipStream_t s) {
    return on_stream("seeds", s, 0);
}
hipError_t launch_gradients(const float*, float4*, int, int, int, const double*, unsigned int*,
                            hipStream_t s) {
    return on_stream("gradients", s, 0, kTables);
}
}  // namespace phx
