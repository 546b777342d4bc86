// A stand-in for the HIP calls that liblinprim.so makes, for tests of its host
// code without a GPU: memory is host memory, kernels do not run, but a launch
// of the counts' read-back is queued (it writes its slot when its stream is
// waited for).  Loaded before the library, so that its names come first.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <vector>

namespace {
struct Slot {
    uint64_t seq, word[2];
};
struct Queued {
    const uint64_t* src;
    int words;
    Slot* slot;
    uint64_t seq;
};
std::vector<Queued> g_queue;
std::vector<const char*> g_names;
std::vector<const void*> g_functions;
alignas(256) int64_t g_symbol[16384];
alignas(64) char g_page[4096];

bool is_read_back(const void* f) {
    for (size_t k = 0; k < g_functions.size(); ++k)
        if (g_functions[k] == f) return strstr(g_names[k], "k_read_back") != nullptr;
    return false;
}
}  // namespace

extern "C" {

// what happened, and what to answer
int fake_host_mallocs, fake_copies, fake_launches, fake_slots_shared;
int fake_pending_error;        // what hipGetLastError answers, once
void (*fake_on_copy)(void);    // called inside a copy, once

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_functions.push_back(f);
    g_names.push_back(name);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}

hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = *block = dim3(1);
    *lds = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipGetDevice(int* dev) {
    *dev = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* prop, int) {
    memset(prop, 0, sizeof(*prop));
    strcpy(prop->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = g_symbol;
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    const int e = fake_pending_error;
    fake_pending_error = 0;
    return (hipError_t)e;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t, unsigned) {
    ++fake_host_mallocs;
    *p = g_page;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* dev) {
    *dev = 0;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void*) {
    memset(at, 0, sizeof(*at));
    at->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
    ++fake_launches;
    if (!is_read_back(f)) return hipSuccess;
    Queued q = {*(const uint64_t**)args[0], *(int*)args[1], *(Slot**)args[2], *(uint64_t*)args[3]};
    for (const Queued& other : g_queue)
        if (other.slot == q.slot) ++fake_slots_shared;
    g_queue.push_back(q);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) {
    ++fake_copies;
    memcpy(dst, src, bytes);
    if (fake_on_copy) {
        void (*f)(void) = fake_on_copy;
        fake_on_copy = nullptr;
        f();
    }
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    for (const Queued& q : g_queue) {
        for (int k = 0; k < q.words; ++k) q.slot->word[k] = q.src[k];
        std::atomic_thread_fence(std::memory_order_release);
        q.slot->seq = q.seq;
    }
    g_queue.clear();
    return hipSuccess;
}
}
