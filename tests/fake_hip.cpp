// A HIP runtime on host memory, for tests of the library's host side without a
// GPU: loaded before libcutgraph.so with its symbols global, it takes the place
// of the runtime the library links.  Allocations are host memory under a limit,
// copies are copies, kernels are not run: every launch, event and stream call is
// written to a log that the test reads.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <dlfcn.h>

#include <cstdio>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <set>
#include <string>
#include <system_error>

static std::map<const void*, std::string> names;   // kernel stubs
static std::map<char*, size_t> blocks;             // live allocations
static size_t used = 0, limit = (size_t)288 << 30, left = ~(size_t)0;
static hipError_t last = hipSuccess;
static std::string text;
static std::set<void*> capturing;
static int64_t next_id = 0x1000;

static hipError_t ret(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}

static void log(const std::string& s) { text += s + "\n"; }

static std::string id(const void* p) {
    char b[32];
    std::snprintf(b, sizeof b, "%llx", (unsigned long long)(uintptr_t)p);
    return b;
}

extern "C" {

// ------------------------------------------------------------- test control --
const char* fake_log() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_limit(size_t bytes) { limit = bytes; }
size_t fake_used() { return used; }
void fake_left(size_t bytes) { left = bytes; }
void fake_capturing(void* stream, int on) {
    if (on) capturing.insert(stream);
    else capturing.erase(stream);
}
// bytes of the allocation that starts at p (0: none)
size_t fake_block(void* p) {
    auto it = blocks.find((char*)p);
    return it == blocks.end() ? 0 : it->second;
}

// threads that may still be started (< 0: any number)
static int threads_left = -1;
void fake_threads(int n) { threads_left = n; }
#define THREAD_START "_ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE"
void fake_start_thread(void* self, void* state, void (*depend)()) asm(THREAD_START);
void fake_start_thread(void* self, void* state, void (*depend)()) {
    if (threads_left == 0) throw std::system_error(EAGAIN, std::generic_category(), "no thread");
    if (threads_left > 0) --threads_left;
    ((void (*)(void*, void*, void (*)()))dlsym(RTLD_NEXT, THREAD_START))(self, state, depend);
}

// ------------------------------------------------------------- registration --
void** __hipRegisterFatBinary(const void*) { return (void**)1; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* device, const char*, unsigned, void*, void*, void*, void*,
                           int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    names[host] = st == 0 && d ? d : device;
    std::free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    cfg_grid = g, cfg_block = b, cfg_lds = lds, cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
    *g = cfg_grid, *b = cfg_block, *lds = cfg_lds, *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t s) {
    std::string n = names[f];
    n = n.substr(0, n.find('('));
    if (n.rfind("void ", 0) == 0) n = n.substr(5);
    if (n.rfind("cut::", 0) == 0) n = n.substr(5);
    log("kernel " + id(s) + " " + std::to_string(g.x) + " " + n);
    return hipSuccess;
}

// ------------------------------------------------------------------- memory --
hipError_t hipMalloc(void** p, size_t n) {
    if (used + n > limit) {
        log("refused " + std::to_string(n));
        *p = nullptr;
        return ret(hipErrorOutOfMemory);
    }
    void* m = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return ret(hipErrorOutOfMemory);
    blocks[(char*)m] = n;
    used += n;
    *p = m;
    log("malloc " + std::to_string(n));
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    auto it = blocks.find((char*)p);
    if (it == blocks.end()) return ret(hipErrorInvalidValue);
    munmap(p, it->second ? it->second : 1);
    used -= it->second;
    log("free " + std::to_string(it->second));
    blocks.erase(it);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
    *f = limit > used ? limit - used : 0;
    if (left < *f) *f = left;
    *t = limit;
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = (void*)0x7000;
    return hipSuccess;
}

// ------------------------------------------------------------------- device --
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 163840;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

// ------------------------------------------------------- streams and events --
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)(next_id += 16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    log("wait " + id(s) + " " + id(e));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)(next_id += 16);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    log("record " + id(s) + " " + id(e));
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}

// ------------------------------------------------------------------- graphs --
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    log("capture " + id(s));
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = (hipGraph_t)(next_id += 16);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = (hipGraphExec_t)(next_id += 16);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
