// A stand-in for the HIP runtime, for host-side tests without a GPU: memory is the
// host's, kernels do not run (their names and launch shapes are recorded), and
// what stream and event queries return is set by the test.  A copy of the solver's
// device state to the host delivers the state that the test set.
#include "nps_internal.hpp"

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {

hipError_t g_query[2] = {hipSuccess, hipSuccess};   // events, streams
nps::State g_state = {};
std::map<const void*, std::string> g_names;
std::string g_launched;                             // "name threads-in-x blocks-in-y\n" per launch
struct {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
} g_config;

}  // namespace

extern "C" {

void fake_query(int stream, int status) { g_query[stream] = static_cast<hipError_t>(status); }
void fake_state(double bb, int n_fluid, int bad_label, int nonfinite) {
    g_state = nps::State{};
    g_state.bb = bb;
    g_state.n_fluid = n_fluid;
    g_state.nlive = 1;
    g_state.bad_label = bad_label;
    g_state.nonfinite = nonfinite;
}
const char* fake_launched() { return g_launched.c_str(); }
void fake_forget() { g_launched.clear(); }

void** __hipRegisterFatBinary(const void*) {
    static void* h = nullptr;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
    g_config = {grid, block, shmem, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *shmem = g_config.shmem;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
    g_launched += g_names[f] + " " + std::to_string((unsigned long long)grid.x * block.x) + " " + std::to_string(grid.y) + "\n";
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "set by the test"; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 4;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (kind == hipMemcpyDeviceToHost && n == sizeof(nps::State)) std::memcpy(dst, &g_state, n);
    else if (kind == hipMemcpyHostToDevice) std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(&g_config);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return g_query[1]; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(&g_config);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return g_query[0]; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}

}  // extern "C"
