// The HIP runtime calls of libgpspca.so without a GPU: launches are recorded and
// not run, device memory is never touched, and a copy to the host delivers the
// control block that the test has set (zeros for anything else).  Loaded before
// the library into the global symbol scope of a child process, so the host code
// under test is the built library's own.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../paper_1312_6182_amd/csrc/gpspca_internal.h"

namespace {

struct State {
    std::mutex mu;
    std::map<const void*, std::string> names;
    std::string log;
    int cus = 256, masked = 0;   // CUs of the device; of them closed to every stream
    gpspca::Ctrl ctrl;
    float first_ms = 1.f, later_ms = 1.f;     // measured times: the first one, the others
    void (*on_sync)(hipStream_t) = nullptr;   // called by hipStreamSynchronize
};
struct Pushed {   // the thread's configuration between push and pop
    dim3 grid, block;
    size_t shm;
    hipStream_t stream;
};
thread_local Pushed t_pushed;
State& S() {
    static State* s = new State;
    return *s;
}

hipError_t record(const void* f, dim3 g, dim3 b, void** args, size_t shm, hipStream_t st) {
    std::lock_guard<std::mutex> lk(S().mu);
    const auto it = S().names.find(f);
    const std::string name = it == S().names.end() ? "?" : it->second;
    char line[512];
    // the column count of a quantizer launch (its fourth argument), else 0
    const long long n = name.find("k_quantize") != std::string::npos
                            ? (long long)*static_cast<int64_t*>(args[3]) : 0;
    std::snprintf(line, sizeof(line), "%s %u %u %u %u %lld %p %lld\n", name.c_str(), g.x, g.y, g.z,
                  b.x * b.y * b.z, (long long)shm, (void*)st, n);
    S().log += line;
    return hipSuccess;
}

}  // namespace

extern "C" {

// ---- what the test sets and reads
void stub_device(int cus, int masked) {
    S().cus = cus;
    S().masked = masked;
}
void stub_result(int n_iter, int status, int abort) {
    std::lock_guard<std::mutex> lk(S().mu);
    std::memset(&S().ctrl, 0, sizeof(gpspca::Ctrl));
    S().ctrl.done = 1;
    S().ctrl.n_iter = n_iter;
    S().ctrl.status = status;
    S().ctrl.abort = abort;
}
void stub_times(float first, float later) {
    S().first_ms = first;
    S().later_ms = later;
}
void stub_on_sync(void (*f)(hipStream_t)) { S().on_sync = f; }
size_t stub_log(char* out, size_t len) {
    std::lock_guard<std::mutex> lk(S().mu);
    std::snprintf(out, len, "%s", S().log.c_str());
    const size_t n = S().log.size();
    if (n < len) S().log.clear();
    return n;
}

// ---- module registration and launches
void** __hipRegisterFatBinary(const void*) { return new void*(nullptr); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
    std::lock_guard<std::mutex> lk(S().mu);
    S().names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t st) {
    t_pushed = Pushed{g, b, shm, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, hipStream_t* st) {
    *g = t_pushed.grid;
    *b = t_pushed.block;
    *shm = t_pushed.shm;
    *st = t_pushed.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shm, hipStream_t st) {
    return record(f, g, b, args, shm, st);
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shm,
                              hipStream_t st, hipEvent_t, hipEvent_t, int) {
    return record(f, g, b, args, shm, st);
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 4;
    return hipSuccess;
}

// ---- device, memory, streams
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = S().cus; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)(uintptr_t)4096; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
    if (k != hipMemcpyDeviceToHost) return hipSuccess;
    std::lock_guard<std::mutex> lk(S().mu);
    if (n == sizeof(gpspca::Ctrl)) std::memcpy(dst, &S().ctrl, n);
    else std::memset(dst, 0, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) {
    if (S().on_sync) S().on_sync(st);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(uintptr_t)64; return hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t st, uint32_t words, uint32_t* mask) {
    // the runtime takes these two for addresses here
    if (st == hipStreamLegacy || st == hipStreamPerThread) std::abort();
    std::memset(mask, 0, 4 * words);
    for (int c = S().masked; c < S().cus && c < 32 * (int)words; ++c) mask[c / 32] |= 1u << (c % 32);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }

// ---- events and graphs
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(uintptr_t)64; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = S().first_ms;
    S().first_ms = S().later_ms;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
