// Drives lagom_overlap_run on a model of the runtime, without a GPU: the HIP entry points that the library calls are defined here and
// found before the real ones.  Streams are clocks in virtual time, a launch moves its stream's clock by the kernel's duration, an
// event is the clock of the stream that recorded it.  The host's clock stands still but for its waits; nothing begins before it was queued.
//   runner_host <fail> <comm us> <comp us> <warmup> <iters> <mode>
// Call <fail> of hipEventElapsedTime fails (0: none).  Prints what the runner returned and measured, and counts what must not happen.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>
#include "lagom.h"

namespace {
struct Event { double at = -1.0; };
struct Op { int stream; bool gate; double begin, end; };
std::map<const void*, std::string>& names() { static auto* m = new std::map<const void*, std::string>; return *m; }     // the library registers its kernels before main's file is initialised
std::map<hipStream_t, double> clock_of;
std::map<hipStream_t, int> queued;                       // operations behind the last synchronisation
std::set<Event*> alive;
std::vector<Op> ops;
int reads = 0, fail_at = 0, created = 0, destroyed_in_flight = 0, ahead = 0;
double comm_us = 1.0, comp_us = 1.0, host = 0.0;
hipStream_t sa = reinterpret_cast<hipStream_t>(16), sb = reinterpret_cast<hipStream_t>(32);
double& queue(hipStream_t st) { ++queued[st]; double& c = clock_of[st]; if (host > c) c = host; return c; }
void wait_until(double at) { if (at > host) host = at; }
bool idle() { return !queued[sa] && !queued[sb]; }
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module = nullptr; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t st);
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t* st);
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = aligned_alloc(64, (n + 63) / 64 * 64); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { Event* x = new Event; alive.insert(x); ++created; *e = reinterpret_cast<hipEvent_t>(x); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { if (!idle()) ++destroyed_in_flight; Event* x = reinterpret_cast<Event*>(e); alive.erase(x); delete x; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) { reinterpret_cast<Event*>(e)->at = queue(st); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
    const double at = reinterpret_cast<Event*>(e)->at;
    double& clock = queue(st);
    if (at > clock) clock = at;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {          // a stream whose clock has not moved since is idle
    wait_until(reinterpret_cast<Event*>(e)->at);
    for (auto& [st, n] : queued) if (clock_of[st] <= reinterpret_cast<Event*>(e)->at) n = 0;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) { wait_until(clock_of[st]); queued[st] = 0; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    if (++reads == fail_at) return hipErrorInvalidHandle;
    *ms = (float)((reinterpret_cast<Event*>(b)->at - reinterpret_cast<Event*>(a)->at) / 1000.0);
    return hipSuccess;
}
static dim3 g_grid, g_block; static size_t g_lds; static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) { g_grid = g; g_block = b; g_lds = s; g_stream = st; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) { *g = g_grid; *b = g_block; *s = g_lds; *st = g_stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t st) {
    const std::string& name = names()[f];
    auto has = [&](const char* s) { return name.find(s) != std::string::npos; };
    if (has("meet_second")) {                           // the probe of the two streams: they meet
        unsigned long long* word = *static_cast<unsigned long long**>(args[0]);
        word[1] = *static_cast<unsigned long long*>(args[1]);
    }
    if (has("gate_leader") && !idle()) ++ahead;         // a repetition that is queued while another one runs
    const bool gate = has("gate_") || has("meet_");
    double& clock = queue(st);
    const double begin = clock;
    clock += gate ? 1.0 : has("gemm") ? comp_us : comm_us;
    ops.push_back({st == sa ? 0 : 1, gate, begin, clock});
    return hipSuccess;
}
}  // extern "C"

int main(int argc, char** argv) {
    if (argc != 7) return 2;
    fail_at = atoi(argv[1]); comm_us = atof(argv[2]); comp_us = atof(argv[3]);
    const int warmup = atoi(argv[4]), iters = atoi(argv[5]), mode = atoi(argv[6]);
    alignas(64) static char memory[6][64];
    const void* srcs[2] = {memory[0], memory[1]};
    void* dsts[1] = {memory[2]};
    lagom_comm_desc comm{};
    comm.op = LAGOM_REDUCE_COPY; comm.dtype = LAGOM_F32; comm.srcs = srcs; comm.nsrc = 2; comm.dsts = dsts; comm.ndst = 1; comm.count = 16; comm.after_comp = -1;
    lagom_gemm_desc comp{};
    comp.A = memory[3]; comp.B = memory[4]; comp.C = memory[5]; comp.M = comp.N = comp.K = 64; comp.b_is_nk = 1; comp.out_dtype = LAGOM_F32; comp.after_comm_id = -1;
    lagom_cfg cfg{4, 256, 65536};
    double x[1], y[1];
    lagom_timing t{};
    t.x_us = x; t.y_us = y;
    const int rc = lagom_overlap_run(&comm, 1, &cfg, 1, &comp, 1, sa, sb, warmup, iters, mode, &t);
    // kernels of one repetition on either stream begin when those of the one before have ended on both
    int comms = 0, comps = 0, early = 0;
    double ended[2] = {0.0, 0.0}, ends = 0.0;
    int seen[2] = {0, 0};
    for (const Op& o : ops) {
        if (o.gate) continue;
        ++(o.stream ? comps : comms);
        if (mode == LAGOM_CORUN && seen[o.stream] == seen[!o.stream]) ends = ended[0] > ended[1] ? ended[0] : ended[1];     // the first one of a repetition
        if (o.begin < ends) ++early;
        ++seen[o.stream];
        ended[o.stream] = o.end;
    }
    std::printf("{\"rc\": %d, \"error\": \"%s\", \"X\": %.3f, \"Y\": %.3f, \"Z\": %.3f, \"comms\": %d, \"comps\": %d, \"early\": %d, \"ahead\": %d, \"reads\": %d, \"created\": %d, "
                "\"destroyed_in_flight\": %d, \"in_flight\": %d, \"alive\": %zu}\n", rc, rc ? lagom_last_error() : "", t.X_us, t.Y_us, t.Z_us, comms, comps, early, ahead, reads,
                created, destroyed_in_flight, idle() ? 0 : 1, alive.size());
    return 0;
}
