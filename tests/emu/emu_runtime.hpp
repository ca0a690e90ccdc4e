// emu_runtime.hpp -- a HIP runtime on the CPU (test infrastructure only): the library's host code and its
// kernels compile against tests/emu/shim with this header before them, and run without a GPU.
//
// Device memory is shared between processes, with an inaccessible page behind every buffer; streams are
// in order and synchronous. A launch runs its workgroups one after another, highest index first, each
// as lockstep threads; a cooperative launch forks a process per workgroup, so that each has its own LDS.
// What a test may ask for (EmuFaults): a cooperative launch that is refused, one that a workgroup does
// not take part in, one whose run has already failed, and an ordinary launch that fails.
#pragma once

#include <hip/hip_runtime.h>

#include <sched.h>
#include <stddef.h>

template <class T> inline T emu_load(T *p)
{
    sched_yield();                       // a poll gives way to the workgroups it waits for
    return std::atomic_ref<T>(*p).load();
}
#define __hip_atomic_load(p, o, s) emu_load(p)
template <class T> inline T atomicMin(T *p, T v)
{
    std::atomic_ref<T> a(*p);
    T o = a.load();
    while (v < o && !a.compare_exchange_weak(o, v)) {}
    return o;
}
using std::erfc;
using std::exp;
using std::max;

// ---- the runtime's types and calls that the library uses -------------------------------------------
typedef void *hipEvent_t;
typedef void *hipGraphExec_t;
constexpr hipError_t hipErrorOutOfMemory = 2, hipErrorLaunchFailure = 719, hipErrorCooperativeLaunchTooLarge = 720;
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeCooperativeLaunch };
enum { hipFuncAttributeMaxDynamicSharedMemorySize };
enum { hipHostMallocDefault };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone };
struct hipDeviceProp_t { char gcnArchName[256]; };

hipError_t hipMalloc(void **p, size_t n);
hipError_t hipFree(void *p);
hipError_t hipMemcpy(void *d, const void *s, size_t n, int kind);
hipError_t hipMemset(void *d, int v, size_t n);
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s);
hipError_t hipFuncSetAttribute(const void *fn, int what, int value);
hipError_t emu_last_error();
hipError_t emu_cooperative(const void *fn, dim3 g, dim3 b, void **args, unsigned lds);
hipError_t hipDeviceGetAttribute(int *v, int what, int device);
bool emu_launch();                       // an ordinary launch: whether it runs

inline hipError_t hipHostMalloc(void **p, size_t n, int) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
inline hipError_t hipHostFree(void *p) { return free(p), hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int kind, hipStream_t) { return hipMemcpy(d, s, n, kind); }
inline hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
inline hipError_t hipEventCreate(hipEvent_t *e) { return *e = new char, hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { return delete static_cast<char *>(e), hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { return *s = hipStreamCaptureStatusNone, hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
inline hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { return std::strcpy(p->gcnArchName, "gfx950"), hipSuccess; }
inline const char *hipGetErrorString(hipError_t e) { return e == hipErrorCooperativeLaunchTooLarge ? "cooperative launch too large" : "emulated failure"; }
#define hipGetLastError() emu_last_error()

inline void emu_grid(dim3 g, dim3 b, const std::function<void()> &f)
{
    for (unsigned y = 0; y < g.y; ++y)
        for (unsigned x = g.x; x-- > 0;) emu_run_block(static_cast<int>(b.x), x, f, y);
}
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(K, G, B, LDS, S, ...)                                          \
    do {                                                                                  \
        if (emu_launch()) emu_grid(G, B, [&] { (K)(__VA_ARGS__); });                      \
    } while (0)
#define hipLaunchCooperativeKernel(F, G, B, A, LDS, S) emu_cooperative(F, G, B, A, LDS)
