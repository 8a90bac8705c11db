// Prints the kernels that lagom_comm_steps and lagom_gemm launch, without a GPU: the HIP entry points that a launch calls are defined here
// and found before the real ones.  Buffers are addresses that nothing reads.
//   launch_host steps <dtype> <count> <nc> <nt> <chunk bytes> <op>:<sources>-<destinations> ...        (a buffer is a letter)
//   launch_host gemm <M>,<N>,<K>,<b_is_nk>,<out dtype> ...
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
#include "lagom.h"

namespace {
std::map<const void*, std::string>& names() { static auto* m = new std::map<const void*, std::string>; return *m; }
dim3 g_grid, g_block; size_t g_lds; hipStream_t g_stream;
std::vector<void*> buffers(const char* from, const char* to) {
    std::vector<void*> out;
    for (; from < to; ++from) out.push_back(reinterpret_cast<void*>((uintptr_t)(*from - 'a' + 1) << 36));
    return out;
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module = nullptr; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) { g_grid = g; g_block = b; g_lds = s; g_stream = st; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) { *g = g_grid; *b = g_block; *s = g_lds; *st = g_stream; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t, hipStream_t) { std::printf("%s %u %u\n", names()[f].c_str(), g.x, b.x); return hipSuccess; }
}  // extern "C"

int steps(int argc, char** argv) {
    if (argc < 6) return 2;
    std::vector<std::vector<void*>> held;
    std::vector<lagom_comm_step> list;
    for (int i = 5; i < argc; ++i) {
        const char *from = std::strchr(argv[i], ':') + 1, *arrow = std::strchr(from, '-');
        held.push_back(buffers(from, arrow));
        held.push_back(buffers(arrow + 1, arrow + std::strlen(arrow)));
        list.push_back({atoi(argv[i]), nullptr, (int32_t)held[held.size() - 2].size(), nullptr, (int32_t)held.back().size()});
    }
    for (size_t i = 0; i < list.size(); ++i) { list[i].srcs = held[2 * i].data(); list[i].dsts = held[2 * i + 1].data(); }
    lagom_cfg cfg{};
    cfg.nc = atoi(argv[2]); cfg.nt = atoi(argv[3]); cfg.chunk_bytes = atoll(argv[4]);
    return lagom_comm_steps((lagom_dtype)atoi(argv[0]), list.data(), (int)list.size(), atoll(argv[1]), &cfg, nullptr);
}

int gemm(int argc, char** argv) {
    const std::vector<void*> m = buffers("abc", "abc" + 3);
    for (int i = 0; i < argc; ++i) {
        long long M, N, K;
        int nk, out;
        if (std::sscanf(argv[i], "%lld,%lld,%lld,%d,%d", &M, &N, &K, &nk, &out) != 5) return 2;
        if (int rc = lagom_gemm(m[0], m[1], m[2], M, N, K, nk, (lagom_dtype)out, nullptr)) return rc;
    }
    return 0;
}

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    const int rc = argv[1][0] == 's' ? steps(argc - 2, argv + 2) : gemm(argc - 2, argv + 2);
    if (rc) std::fprintf(stderr, "%s\n", lagom_last_error());
    return rc ? 1 : 0;
}
