// A stand-in for the HIP runtime that does no GPU work: it hands out addresses, keeps track of what is allocated and of which
// stream a graph is being recorded on, and writes down every call.  Loaded in front of the library it lets the library's host code
// run, and be looked at, on a machine without a GPU.  (The few types are those of the C interface: 12-byte dim3, int status.)
#include <cxxabi.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <set>
#include <string>

struct Dim3 { uint32_t x, y, z; };
static const int kOk = 0, kInvalid = 1, kOutOfMemory = 2, kNotSupported = 801, kCaptureUnsupported = 900, kCaptureIsolation = 905;
static const int kCanWaitForValues = 10013, kSignalMemory = 2, kRelaxed = 2;

static std::string log_text;
static std::map<uint64_t, size_t> blocks;                 // address -> bytes
static size_t held, limit = ~(size_t)0;
static uint64_t next_address = 0x100000000ull, next_event = 1;
static std::map<const void*, std::string> kernels;
static std::set<void*> capturing, joined_back;            // streams that record a graph; those of them that the origin waits for
static void* origin;
static std::map<void*, std::pair<void*, bool>> events;    // event -> stream it was recorded on, in a graph or not
static struct { Dim3 grid, block; size_t shmem; void* stream; } pushed;
static int capture_mode, refused;                         // of this thread; kinds of value calls that fail (refuse_values)
static bool landing = true;                               // values are written as soon as they are asked for
static std::map<uint64_t*, std::pair<uint64_t, uint64_t>> signals;        // eight bytes that streams write -> values asked for, and there
static size_t in_use() { return held + 8 * signals.size(); }
static bool forbidden() { return !capturing.empty() && capture_mode != kRelaxed; }       // nothing may be allocated: a graph is recorded

template <typename... A> static void note(const char* fmt, A... a) {
    char buf[512];
    snprintf(buf, sizeof(buf), fmt, a...);
    log_text += buf;
    log_text += '\n';
}

extern "C" {

// ---- for the test
const char* recorded() { return log_text.c_str(); }
void forget() { log_text.clear(); }
void limit_memory(size_t bytes) { limit = bytes; }
size_t memory_held() { return in_use(); }
void refuse_values(int kinds) { refused = kinds; }        // 1: the device says it cannot, 2: no memory for them, 4: no write, 8: no wait
void land_values(int on) {                                // off: writes that are asked for from now on are on their way until it is on again
    landing = on != 0;
    if (landing)
        for (auto& s : signals) *s.first = s.second.second = s.second.first;
}
void begin_capture(void* s) { capturing = {s}; joined_back = {s}; origin = s; }
int end_capture() {                                       // streams that were drawn into the graph and not joined back
    int open = 0;
    for (void* s : capturing) open += !joined_back.count(s);
    capturing.clear();
    return open;
}

// ---- the runtime's interface, as far as the library uses it
int hipGetDeviceCount(int* n) { *n = 1; return kOk; }
int hipSetDevice(int) { return kOk; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }
int hipDeviceSynchronize() { note("synchronize"); return capturing.empty() ? kOk : kCaptureUnsupported; }
const char* hipGetErrorString(int) { return "recorded error"; }
int hipGetLastError() { return kOk; }
int hipFuncSetAttribute(const void*, int, int) { return kOk; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x10000000ull; return kOk; }
int hipPointerGetAttributes(int* type, const void*) { *type = 2; return kOk; }       // device memory

int hipMalloc(void** p, size_t bytes) {
    if (forbidden()) { note("malloc in a graph"); return kCaptureUnsupported; }
    if (bytes > limit || in_use() > limit - bytes) { note("no memory %zu", bytes); return kOutOfMemory; }
    *p = (void*)next_address;
    note("malloc %llx %zu", (unsigned long long)next_address, bytes);
    blocks[next_address] = bytes;
    held += bytes;
    next_address += (bytes + 0xFFFFF) & ~0xFFFFFull;
    return kOk;
}
int hipExtMallocWithFlags(void** p, size_t bytes, unsigned flags) {
    if (forbidden()) { note("malloc in a graph"); return kCaptureUnsupported; }
    if (flags != kSignalMemory || bytes != 8) return kInvalid;
    note("malloc signal");
    if ((refused & 2) || bytes > limit || in_use() > limit - bytes) return kOutOfMemory;
    uint64_t* at = new uint64_t(~0ull);
    signals[at] = {0, 0};                                  // (what the library is to store there)
    *p = at;
    return kOk;
}
int hipFree(void* p) {
    if (signals.count((uint64_t*)p)) {
        signals.erase((uint64_t*)p);
        delete (uint64_t*)p;
        note("free signal");
        return kOk;
    }
    note("free %llx", (unsigned long long)(uintptr_t)p);
    held -= blocks[(uint64_t)(uintptr_t)p];
    blocks.erase((uint64_t)(uintptr_t)p);
    return kOk;
}
int hipMemset(void*, int, size_t) { return kOk; }

int hipDeviceGetAttribute(int* value, int attribute, int) {
    *value = attribute == kCanWaitForValues && !(refused & 1);
    return attribute == kCanWaitForValues ? kOk : kInvalid;
}
int hipThreadExchangeStreamCaptureMode(int* mode) { const int was = capture_mode; capture_mode = *mode; *mode = was; return kOk; }
int hipStreamWriteValue64(void* s, void* p, uint64_t value, unsigned) {
    note("write %p %p %llu", s, p, (unsigned long long)value);
    if ((refused & 4) || capturing.count(s)) return kNotSupported;
    const auto at = signals.find((uint64_t*)p);
    if (at == signals.end() || *at->first != at->second.first) return kInvalid;          // one write on its way at most
    at->second.first = value;
    if (landing) *at->first = at->second.second = value;
    return kOk;
}
int hipStreamWaitValue64(void* s, void* p, uint64_t value, unsigned flags, uint64_t mask) {
    note("await %p %p %llu", s, p, (unsigned long long)value);
    if ((refused & 8) || capturing.count(s)) return kNotSupported;
    const auto at = signals.find((uint64_t*)p);                                          // (flags 0: until it is as large)
    return at == signals.end() || at->second.first < value || flags != 0 || mask != ~0ull ? kInvalid : kOk;
}
int hipStreamIsCapturing(void* s, int* status) { *status = capturing.count(s) ? 1 : 0; return kOk; }
int hipStreamSynchronize(void*) { return kOk; }
int hipStreamDestroy(void*) { return kOk; }
int hipExtStreamCreateWithCUMask(void** s, uint32_t, const uint32_t*) { *s = (void*)(0xABC000 + next_event++); return kOk; }
int hipEventCreate(void** e) { *e = (void*)next_event++; return kOk; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)next_event++; return kOk; }
int hipEventDestroy(void*) { return kOk; }
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return kOk; }
int hipEventRecord(void* e, void* s) {
    note("record %p %p", e, s);
    events[e] = {s, capturing.count(s) != 0};
    return kOk;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) {
    note("wait %p %p", s, e);
    const auto at = events[e];
    if (capturing.count(s) && !at.second) return kCaptureIsolation;        // a wait that leads out of the graph
    if (at.second) capturing.insert(s);
    if (s == origin && at.second) joined_back.insert(at.first);
    return kOk;
}

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shmem, void* s) { pushed = {grid, block, shmem, s}; return kOk; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shmem, void** s) {
    *grid = pushed.grid; *block = pushed.block; *shmem = pushed.shmem; *s = pushed.stream;
    return kOk;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t shmem, void* s) {
    note("launch %s %u %u %u %zu %p", kernels[f].c_str(), grid.x, grid.y, block.x, shmem, s);
    return kOk;
}
void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string n = plain ? plain : name;                 // "void (anonymous namespace)::k_name<args>(types)" -> "k_name<args>"
    free(plain);
    const size_t at = n.find("k_");
    size_t end = at == std::string::npos ? at : n.find('(', at);
    while (end != std::string::npos && n.compare(end, 12, "(anonymous n") == 0) end = n.find('(', end + 12);   // a template argument's
    n = at == std::string::npos ? n : n.substr(at, end - at);
    for (size_t sp; (sp = n.find(' ')) != std::string::npos;) n.erase(sp, 1);
    kernels[f] = n;
}

}
