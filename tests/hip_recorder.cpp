// Host-only stand-in for the HIP runtime calls of libprony, and a driver that runs the
// C ABI on it: allocations are reserved addresses (under a limit that a scenario sets),
// launches are recorded by kernel name and run nothing. Commands come from stdin, one
// per line; each prints "<status> <allocations> <bytes held> <kernels launched>".
// The definitions here take the place of libamdhip64's (the executable comes first in
// the dynamic symbol order).
#include <algorithm>

#include <cxxabi.h>
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "prony.h"

namespace {

std::map<const void*, std::string>& kernels() {      // host function -> kernel name
    static std::map<const void*, std::string> k;
    return k;
}
std::map<void*, size_t> held;
size_t held_bytes = 0, limit = SIZE_MAX;
int allocations = 0;
bool capturing = false;
std::vector<std::string> launched;
hipError_t last = hipSuccess;

std::string base_name(const char* mangled) {
    int status = 0;
    char* d = abi::__cxa_demangle(mangled, nullptr, nullptr, &status);
    std::string s = status == 0 ? d : mangled;
    free(d);
    if (s.rfind("void ", 0) == 0) s = s.substr(5);
    size_t at;
    while ((at = s.find("prony::")) != std::string::npos) s.erase(at, 7);
    while ((at = s.find("(anonymous namespace)::")) != std::string::npos) s.erase(at, 23);
    s = s.substr(0, s.find('('));
    s.erase(std::remove(s.begin(), s.end(), ' '), s.end());
    return s;
}

hipError_t ok(hipError_t e = hipSuccess) {
    if (e != hipSuccess) last = e;
    return e;
}

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    kernels()[host] = base_name(name);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
    config = {g, b, s, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
    *g = config.grid, *b = config.block, *s = config.shared, *st = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t shared, hipStream_t) {
    if (!g.x || !g.y || !g.z || b.x > 1024 || shared > 160 * 1024) return ok(hipErrorInvalidValue);
    launched.push_back(kernels()[f]);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (capturing) return ok(hipErrorStreamCaptureUnsupported);
    if (n > limit - std::min(limit, held_bytes)) return ok(hipErrorOutOfMemory);
    // addresses only: no kernel runs and no copy is made
    *p = mmap(nullptr, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) return ok(hipErrorOutOfMemory);
    held[*p] = n;
    held_bytes += n;
    ++allocations;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    munmap(p, held[p]);
    held_bytes -= held[p];
    held.erase(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "recorded error"; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = p->maxSharedMemoryPerMultiProcessor = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char scratch[1];
    *p = scratch;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int v) {
    return v <= 160 * 1024 ? hipSuccess : ok(hipErrorInvalidValue);
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(&config);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(&config);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
}

int main() {
    prony_handle_t h = nullptr;
    prony_factors_t factors = nullptr;
    prony_batch_t batch = nullptr;
    double* const p = reinterpret_cast<double*>(0x1000);   // never dereferenced
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string what;
        in >> what;
        std::vector<long long> a;
        for (long long v; in >> v;) a.push_back(v);
        a.resize(std::max<size_t>(a.size(), 8));
        const int d = (int)a[0], n = (int)a[1], m = (int)a[2];
        const auto prec = (prony_prec_t)a[3];
        const int before = allocations;
        launched.clear();
        int st = -1;
        if (what == "create") st = prony_create(&h, 0);
        else if (what == "destroy") st = prony_destroy(h);
        else if (what == "limit") limit = (size_t)a[0], st = 0;      // bytes that may be held
        else if (what == "capture") capturing = a[0], st = 0;
        else if (what == "reserve") st = prony_reserve(h, d, n, m);
        else if (what == "tune") st = prony_tune_set_tile(h, d, n, m, prec, 0, (int)a[4], (int)a[5]);
        else if (what == "plan") {
            size_t bytes = 0;
            st = prony_build_S_plan(h, d, n, m, prec, (unsigned)a[4], nullptr, nullptr, nullptr, &bytes);
            std::cout << bytes << " ";
        }
        else if (what == "build") st = prony_build_S(h, d, n, m, p, p, m, 1, p, p, m, 1, prec, (unsigned)a[4], p);
        else if (what == "noalloc")
            st = prony_build_S_noalloc(h, d, n, m, p, p, m, 1, p, p, m, 1, prec, (unsigned)a[4], p);
        else if (what == "adjoint") st = prony_build_S_adjoint(h, d, n, m, p, m, 1, p, p, m, 1, p, prec, p);
        else if (what == "product") st = prony_toeplitz_mm(h, d, n, (int)a[4], p, m, p, m, prec, p, m);
        else if (what == "coeffs") st = prony_coeffs(h, d, n, m, p, p, p, p, a[3] ? p : nullptr);
        else if (what == "factors")
            st = prony_factors_create(h, d, n, m, p, m, 1, p, p, m, 1, prec, (unsigned)a[4], &factors);
        else if (what == "build_factors") st = prony_build_S_factors(h, factors, p, p);
        else if (what == "free_factors") st = prony_factors_destroy(factors);
        else if (what == "batch") {                                  // prec, then d n m of every instance
            std::vector<prony_instance_t> inst;
            for (size_t i = 1; i + 2 < a.size() && a[i]; i += 3)
                inst.push_back({(int)a[i], (int)a[i + 1], (int)a[i + 2], p, p, p, p, p});
            st = prony_batch_create(h, (int)inst.size(), inst.data(), (prony_prec_t)a[0], &batch);
        }
        else if (what == "run_batch") st = prony_build_S_batched(h, batch);
        else if (what == "adjoint_batch") st = prony_build_S_adjoint_batched(h, batch, p, p);
        else if (what == "free_batch") st = prony_batch_destroy(batch);
        std::cout << st << " " << allocations - before << " " << held_bytes;
        for (const auto& k : launched) std::cout << " " << k;
        std::cout << "\n";
    }
    return 0;
}
