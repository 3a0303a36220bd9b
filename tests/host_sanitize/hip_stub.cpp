// Stand-in for the HIP runtime, for a host-only build of the library under AddressSanitizer and
// UndefinedBehaviorSanitizer (CPU only).  "Device" and pinned memory are ordinary heap blocks of
// exactly the requested size, so that every table the planner fills and every copy it enqueues is
// checked against the size it allocated; copies and fills happen at once; kernel launches do
// nothing, but that those which send a call's result to pinned host memory send "no error, empty
// message" with the call's number (or, if the test says so, end without it, as a kernel does that
// finds an invariant violated); streams and events are inert, but that one stream can be made one that has been
// destroyed, one that records a graph, and events ones that have not happened.  One device.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>

static long g_launches = 0;
static unsigned g_grids[64];           // workgroups (x) of the latest launches
static size_t g_lds[64];               // their dynamic LDS
static const void* g_kernels[64];      // and their kernels
static long g_live_blocks = 0;
static long g_fail_alloc_at = -1;      // the n-th allocation from now fails (tests the clean-up path)
static bool g_withhold = false;        // no results are sent
static uint32_t g_result_bits = 0;     // the error word that results carry
static struct { const char* kernel; uint32_t bits; } g_next[4];          // ... and the next result of kernels with that name
static hipError_t g_launch_error = hipSuccess;
static hipStream_t g_gone = nullptr, g_recording = nullptr;
static bool g_events_pending = false;
static int g_stream_waits = 0, g_event_waits = 0, g_relaxed = 0;
static struct { const void* host; const char* name; } g_names[128];      // every kernel with its mangled name
static int g_n_names = 0;
// The kernels that send results, by a part of their mangled name, and which of their arguments are the word
// in pinned memory and the call's number.
struct Sender { const char* name; int word, seq; const void* host[2]; };
static Sender g_senders[] = {
    {"10k_emit_all", 13, 14, {}}, {"11k_emit_scan", 13, 14, {}}, {"6k_emitILb1E", 18, 19, {}}, {"16k_finish_message", 11, 12, {}}, {"9k_publish", 0, 2, {}}};

extern "C" long stub_launches() { return g_launches; }
extern "C" unsigned stub_grid(long launch) { return g_grids[launch % 64]; }
extern "C" const void* stub_kernel(long launch) { return g_kernels[launch % 64]; }
extern "C" long stub_live_blocks() { return g_live_blocks; }
extern "C" void stub_fail_allocation(long nth) { g_fail_alloc_at = nth; }
extern "C" void stub_withhold_results(int on) { g_withhold = on != 0; }
extern "C" void stub_result_bits(uint32_t bits) { g_result_bits = bits; }
extern "C" void stub_next_result_bits(const char* kernel, uint32_t bits) {
    for (auto& n : g_next)
        if (!n.kernel) { n = {kernel, bits}; return; }
}
// Workgroups (x) of the first of the launches from number `from` on of a kernel with that name (0: none).
extern "C" unsigned stub_grid_of(const char* name, long from) {
    for (long i = from; i < g_launches; ++i)
        for (int k = 0; k < g_n_names; ++k)
            if (g_kernels[i % 64] == g_names[k].host && std::strstr(g_names[k].name, name)) return g_grids[i % 64];
    return 0;
}
// ... and its dynamic LDS.
extern "C" size_t stub_lds_of(const char* name, long from) {
    for (long i = from; i < g_launches; ++i)
        for (int k = 0; k < g_n_names; ++k)
            if (g_kernels[i % 64] == g_names[k].host && std::strstr(g_names[k].name, name)) return g_lds[i % 64];
    return 0;
}
// How many of the launches from number `from` on (of the latest 64) were of kernels with that name.
extern "C" int stub_launched(const char* name, long from) {
    int n = 0;
    for (long i = from; i < g_launches; ++i)
        for (int k = 0; k < g_n_names; ++k)
            n += g_kernels[i % 64] == g_names[k].host && std::strstr(g_names[k].name, name);
    return n;
}
extern "C" void stub_stream_gone(void* s) { g_gone = (hipStream_t)s; }
extern "C" void stub_stream_records(void* s) { g_recording = (hipStream_t)s; }
extern "C" void stub_events_pending(int on) { g_events_pending = on != 0; }
extern "C" int stub_stream_waits() { return g_stream_waits; }
extern "C" int stub_event_waits() { return g_event_waits; }
extern "C" int stub_known_senders() {
    int n = 0;
    for (const Sender& s : g_senders) n += (s.host[0] != nullptr) + (s.host[1] != nullptr);
    return n;
}

static hipError_t stub_alloc(void** p, size_t bytes) {
    if (!p) return hipErrorInvalidValue;
    if (g_fail_alloc_at >= 0 && g_fail_alloc_at-- == 0) { *p = nullptr; return hipErrorOutOfMemory; }
    *p = std::calloc(bytes ? bytes : 1, 1);          // (zero-filled: a result block no kernel wrote reads "no error")
    if (!*p) return hipErrorOutOfMemory;
    ++g_live_blocks;
    return hipSuccess;
}
static hipError_t stub_free(void* p) {
    if (p) { std::free(p); --g_live_blocks; }
    return hipSuccess;
}

extern "C" {

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : hipErrorInvalidDevice; }
hipError_t hipGetLastError(void) { const hipError_t e = g_launch_error; g_launch_error = hipSuccess; return e; }

hipError_t hipMalloc(void** p, size_t bytes) { return stub_alloc(p, bytes); }
hipError_t hipFree(void* p) { return stub_free(p); }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int) { return stub_alloc(p, bytes); }
hipError_t hipHostFree(void* p) { return stub_free(p); }
hipError_t hipHostGetDevicePointer(void** dev, void* host, unsigned int) { *dev = host; return hipSuccess; }

hipError_t hipMemcpy(void* dst, const void* src, size_t bytes, hipMemcpyKind) { if (bytes) std::memcpy(dst, src, bytes); return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t s) {
    if (s && s == g_gone) return hipErrorContextIsDestroyed;
    if (bytes) std::memcpy(dst, src, bytes);
    return hipSuccess;
}
hipError_t hipMemset(void* dst, int value, size_t bytes) { if (bytes) std::memset(dst, value, bytes); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return s && s == g_gone ? hipErrorContextIsDestroyed : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
    *status = s && s == g_recording ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* mode) {
    g_relaxed += *mode == hipStreamCaptureModeRelaxed ? 1 : -1;
    *mode = g_relaxed ? hipStreamCaptureModeGlobal : hipStreamCaptureModeRelaxed;
    return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t* e) { return stub_alloc(reinterpret_cast<void**>(e), 8); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return stub_alloc(reinterpret_cast<void**>(e), 8); }
hipError_t hipEventDestroy(hipEvent_t e) { return stub_free(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { ++g_event_waits; return g_recording && !g_relaxed ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) {
    if (g_recording && !g_relaxed) return hipErrorStreamCaptureUnsupported;
    return g_events_pending ? hipErrorNotReady : hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
    ++g_stream_waits;
    return s && s == g_recording ? hipErrorStreamCaptureIsolation : hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t) {
    // (as the runtime does: at most 2^32 - 1 work items in a dimension)
    if (grid.x == 0 || grid.y == 0 || grid.z == 0 || block.x == 0 || block.x * block.y * block.z > 1024 ||
        (uint64_t)grid.x * block.x > 0xFFFFFFFFull || grid.y > 65535u || grid.z > 65535u)
        return g_launch_error = hipErrorInvalidConfiguration;
    for (const Sender& s : g_senders)
        if ((f == s.host[0] || f == s.host[1]) && !g_withhold) {     // (the number: bits 50 to 63 of the word)
            uint32_t bits = g_result_bits;
            for (auto& n : g_next)
                if (n.kernel && std::strstr(s.name, n.kernel)) { bits = n.bits; n.kernel = nullptr; break; }
            **static_cast<uint64_t**>(args[s.word]) = (uint64_t)(*static_cast<uint32_t*>(args[s.seq]) & 0x3FFFu) << 50 |
                                                      (uint64_t)bits << 40;
        }
    g_grids[g_launches % 64] = grid.x;
    g_lds[g_launches % 64] = shmem;
    g_kernels[g_launches++ % 64] = f;
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t s, hipEvent_t,
                              hipEvent_t, int) {
    return hipLaunchKernel(f, grid, block, args, shmem, s);
}
// the host-side shadow of a device variable has the variable's size: it serves as its storage
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = const_cast<void*>(symbol); return hipSuccess; }

// what the compiler-generated registration code calls
void** __hipRegisterFatBinary(const void*) { static void* handle = nullptr; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    if (g_n_names < 128) g_names[g_n_names++] = {host, name};
    for (Sender& s : g_senders)
        if (std::strstr(name, s.name)) s.host[s.host[0] ? 1 : 0] = host;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static dim3 g_grid, g_block;
static size_t g_shmem;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
    g_grid = grid; g_block = block; g_shmem = shmem; g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
    *grid = g_grid; *block = g_block; *shmem = g_shmem; *s = g_stream;
    return hipSuccess;
}

}  // extern "C"
