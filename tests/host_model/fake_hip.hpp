// The HIP runtime calls that libround_attention.so makes, on two devices that are not there: a program that includes this file
// and is linked (with -rdynamic) against the library runs its host code on the CPU.  Memory is host memory and kernels are
// only noted; every call that enqueues something is noted with the device of its stream.  Include it once.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace fake {
constexpr int kDevices = 2;
struct Stream {
    int device;
};
struct Event {
    int device;
};
struct Op {
    std::string what;  // "kernel", "copy", "wait", "record"
    std::string name;  // of the kernel
    int device;        // of the stream
    dim3 grid, block;
    const char *dst, *src;
    size_t bytes;
    hipStream_t stream;
    hipEvent_t event;
};
struct Allocation {
    size_t bytes;
    unsigned flags;
    bool host;
};
struct State {
    int current = 0;
    std::vector<Op> ops;
    std::map<uintptr_t, Allocation> memory;
    std::map<const void*, std::string> kernels;
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
inline State& state() {
    static State s;
    return s;
}
inline bool is_default(hipStream_t st) { return st == nullptr || st == hipStreamLegacy || st == hipStreamPerThread; }
inline int device_of(hipStream_t st) { return is_default(st) ? state().current : reinterpret_cast<Stream*>(st)->device; }
inline hipStream_t handle(Stream& s) { return reinterpret_cast<hipStream_t>(&s); }
inline void note(Op op) { state().ops.push_back(op); }
inline void* allocate(size_t bytes, unsigned flags, bool host) {
    void* p = nullptr;
    if (posix_memalign(&p, 4096, bytes ? bytes : 1)) return nullptr;
    state().memory[reinterpret_cast<uintptr_t>(p)] = {bytes, flags, host};
    return p;
}
// An allocation at a given place of memory that the program owns.
inline void place(void* p, size_t bytes, unsigned flags) { state().memory[reinterpret_cast<uintptr_t>(p)] = {bytes, flags, true}; }
inline const std::pair<const uintptr_t, Allocation>* find(const void* p) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(p);
    auto it = state().memory.upper_bound(x);
    if (it == state().memory.begin()) return nullptr;
    --it;
    return x < it->first + it->second.bytes ? &*it : nullptr;
}
// Whether op j is ordered behind op i: the same stream, or over events recorded behind it and waited for.
inline bool before(const std::vector<Op>& ops, size_t i, size_t j) {
    std::vector<hipStream_t> streams{ops[i].stream};
    std::vector<hipEvent_t> events;
    auto has = [](const auto& v, auto x) {
        for (auto y : v)
            if (y == x) return true;
        return false;
    };
    for (size_t k = i + 1; k <= j; ++k) {
        if (ops[k].what == "wait" && has(events, ops[k].event) && !has(streams, ops[k].stream)) streams.push_back(ops[k].stream);
        if (ops[k].what == "record") {
            for (size_t e = 0; e < events.size();) {  // recorded anew
                if (events[e] == ops[k].event) events.erase(events.begin() + e);
                else ++e;
            }
            if (has(streams, ops[k].stream)) events.push_back(ops[k].event);
        }
    }
    return has(streams, ops[j].stream);
}
// Whether a wait for `event` behind all of the ops covers op i.
inline bool reaches(std::vector<Op> ops, hipEvent_t event, size_t i) {
    static Stream probe{0};
    ops.push_back({"wait", "", 0, {}, {}, nullptr, nullptr, 0, handle(probe), event});
    return before(ops, i, ops.size() - 1);
}
// Whether what is enqueued next on `st` comes behind op i.
inline bool reaches_end(std::vector<Op> ops, hipStream_t st, size_t i) {
    ops.push_back({"next", "", 0, {}, {}, nullptr, nullptr, 0, st, nullptr});
    return before(ops, i, ops.size() - 1);
}
inline int count(const char* what) {
    int n = 0;
    for (const Op& op : state().ops) n += op.what == what;
    return n;
}
}  // namespace fake

extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = fake::kDevices, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = fake::state().current, hipSuccess; }
hipError_t hipSetDevice(int d) {
    if (d < 0 || d >= fake::kDevices) return hipErrorInvalidDevice;
    return fake::state().current = d, hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return (*p = fake::allocate(n, 0, false)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) { return (*p = fake::allocate(n, flags, true)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) {
    fake::state().memory.erase(reinterpret_cast<uintptr_t>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { return *p = const_cast<void*>(symbol), hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    const auto* m = fake::find(p);
    if (!m) return hipErrorInvalidValue;
    std::memset(a, 0, sizeof(*a));
    a->type = m->second.host ? hipMemoryTypeHost : hipMemoryTypeDevice;
    a->devicePointer = const_cast<void*>(p);
    a->hostPointer = m->second.host ? const_cast<void*>(p) : nullptr;
    a->allocationFlags = m->second.flags;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* bytes, hipDeviceptr_t p) {
    const auto* m = fake::find(p);
    if (!m) return hipErrorNotFound;
    *base = reinterpret_cast<void*>(m->first);
    *bytes = m->second.bytes;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t st, hipDevice_t* d) {  // (the runtime's reads what the handle points to)
    return *d = st == nullptr ? fake::state().current : reinterpret_cast<fake::Stream*>(st)->device, hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new fake::Event{fake::state().current});
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete reinterpret_cast<fake::Event*>(e), hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
    if (reinterpret_cast<fake::Event*>(e)->device != fake::device_of(st)) return hipErrorInvalidHandle;
    fake::note({"record", "", fake::device_of(st), {}, {}, nullptr, nullptr, 0, st, e});
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
    fake::note({"wait", "", fake::device_of(st), {}, {}, nullptr, nullptr, 0, st, e});
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t st) {
    fake::note({"copy", "", fake::device_of(st), {}, {}, static_cast<const char*>(dst), static_cast<const char*>(src), n, st, nullptr});
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t st) {
    fake::note({"kernel", fake::state().kernels[f], fake::device_of(st), grid, block, nullptr, nullptr, 0, st, nullptr});
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t st, hipEvent_t, hipEvent_t, int) {
    return hipLaunchKernel(f, grid, block, args, shared, st);
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorInvalidHandle ? "invalid resource handle" : "error"; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t st) {
    fake::state().grid = grid;
    fake::state().block = block;
    fake::state().shared = shared;
    fake::state().stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* st) {
    *grid = fake::state().grid;
    *block = fake::state().block;
    *shared = fake::state().shared;
    *st = fake::state().stream;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
    static void* module;
    return &module;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    fake::state().kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}
