// A HIP runtime without a device, for tests of the host code's error paths: memory is host memory, kernels do not run.  Preloaded into a
// process of its own.  FAKE_HIP_FAIL=<function>:<text>:<error>: launches of kernels whose name contains the text ("launch"), or the allocation
// of as many bytes or more as the text says ("malloc"), fail with that error.  The launches are kept (fake_hip_launch).
// FAKE_HIP_SIZES=<up to five numbers, :>: what row_layout_kernel tells the host (csrc/frontend.hip, FrontResult: early and totals).
#define __HIP_PLATFORM_AMD__
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <pthread.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string name;
    unsigned grid[3], threads, lds, args[2];
};
std::vector<Launch>& launches() {
    static std::vector<Launch> l;
    return l;
}
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> n;
    return n;
}
hipError_t g_last = hipSuccess;
hipError_t fail(hipError_t e) { return g_last = e; }
bool wanted(const char* what, std::string* text, hipError_t* error) {
    const char* f = std::getenv("FAKE_HIP_FAIL");
    if (!f) return false;
    const std::string s(f);
    const size_t a = s.find(':'), b = s.rfind(':');
    if (a == std::string::npos || a == b || s.substr(0, a) != what) return false;
    *text = s.substr(a + 1, b - a - 1);
    *error = (hipError_t)std::atoi(s.c_str() + b + 1);
    return true;
}
std::map<void*, size_t>& blocks() {
    static std::map<void*, size_t> b;
    return b;
}
hipError_t get(void** p, size_t bytes) {
    std::string text;
    hipError_t e;
    if (wanted("malloc", &text, &e) && bytes >= std::strtoull(text.c_str(), nullptr, 10)) return fail(e);
    *p = std::calloc(1, bytes + 256);
    blocks()[*p] = bytes;
    return hipSuccess;
}
hipError_t give(void* p) {
    blocks().erase(p);
    std::free(p);
    return hipSuccess;
}
}  // namespace

extern "C" {
size_t fake_hip_bytes() {  // in device memory
    size_t s = 0;
    for (auto& b : blocks()) s += b.second;
    return s;
}
static thread_local int g_started;
int fake_hip_threads() { return g_started; }  // threads that the calling thread has started
int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
    static const auto real = reinterpret_cast<int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*)>(dlsym(RTLD_NEXT, "pthread_create"));
    ++g_started;
    return real(t, a, f, arg);
}
// The latest launch of a kernel whose (mangled) name contains the text: its name, and grid, threads of a workgroup, bytes of dynamic LDS; of
// cer_gemv_tab_kernel the rows per workgroup and `meta` as well.
const char* fake_hip_launch(const char* text, unsigned* shape) {
    for (size_t i = launches().size(); i-- > 0;) {
        const Launch& l = launches()[i];
        if (l.name.find(text) == std::string::npos) continue;
        const unsigned s[7] = {l.grid[0], l.grid[1], l.grid[2], l.threads, l.lds, l.args[0], l.args[1]};
        std::memcpy(shape, s, sizeof s);
        return l.name.c_str();
    }
    return nullptr;
}
void fake_hip_forget() { launches().clear(); }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned int, void*, void*, void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock || a == hipDeviceAttributeSharedMemPerBlockOptin ? 160 * 1024 : 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = p->sharedMemPerBlockOptin = p->maxSharedMemoryPerMultiProcessor = 160 * 1024;
    p->totalGlobalMem = (size_t)288 << 30;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipMalloc(void** p, size_t n) { return get(p, n); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return get(p, n); }
hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t, hipStream_t) { return get(p, n); }
hipError_t hipFree(void* p) { return give(p); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return give(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
    std::string text;
    hipError_t e;
    if (wanted("launch", &text, &e) && names()[f].find(text) != std::string::npos) return fail(e);
    if (const char* words = std::getenv("FAKE_HIP_SIZES"); words && names()[f].find("row_layout_kernel") != std::string::npos) {
        auto* told = *static_cast<unsigned long long**>(args[8]);
        for (int i = 0; i < 5 && *words; ++i) {
            char* end;
            told[i] = std::strtoull(words, &end, 10) | 1ull << 63;
            words = end + (*end == ':');
        }
    }
    Launch l{names()[f], {grid.x, grid.y, grid.z}, block.x, (unsigned)lds, {0, 0}};
    if (l.name.find("cer_gemv_tab_kernel") != std::string::npos)
        for (int i = 0; i < 2; ++i) l.args[i] = *static_cast<unsigned*>(args[7 + i]);
    launches().push_back(l);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { std::memset(a, 0, sizeof *a); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)std::calloc(1, 1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void*)e); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) { *p = (hipMemPool_t)std::calloc(1, 1); return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t p) { std::free((void*)p); return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return hipSuccess; }
}
