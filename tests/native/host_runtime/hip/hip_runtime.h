// A host-only stand-in for the HIP runtime calls that ppd_api.hip makes, for tests on machines without a GPU: memory comes
// from malloc (AddressSanitizer sees every overrun), a stream is a queue of closures that run when something waits for it
// or when the test runs it, kernels run on the CPU.  The test sets what the calls return (`sim`).
#pragma once
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <mutex>

#define __global__
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n((p), (v), (order))
#define HIP_SYMBOL(x) (&(x))

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct alignas(16) uint4 { uint32_t x, y, z, w; };
inline thread_local dim3 blockIdx, threadIdx, blockDim, gridDim;
inline void __syncthreads() {}
inline uint32_t atomicAdd(uint32_t* p, uint32_t v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
inline uint32_t atomicOr(uint32_t* p, uint32_t v) { return __atomic_fetch_or(p, v, __ATOMIC_RELAXED); }
inline uint32_t atomicAnd(uint32_t* p, uint32_t v) { return __atomic_fetch_and(p, v, __ATOMIC_RELAXED); }

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorLaunchFailure = 719, hipErrorNotReady = 600 };
enum hipMemcpyKind { hipMemcpyDeviceToHost };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
constexpr unsigned hipEventDisableTiming = 2, hipStreamNonBlocking = 1, hipHostMallocDefault = 0, hipHostMallocMapped = 2, hipHostMallocCoherent = 0x40000000;
class SimStream {
public:
    void push(std::function<void()> f) {
        std::lock_guard<std::mutex> lock(m_);
        work_.push_back(std::move(f));
    }
    // runs what is enqueued, in order; at most `count` entries
    void run(size_t count = SIZE_MAX) {
        for (; count > 0; --count) {
            std::function<void()> f;
            {
                std::lock_guard<std::mutex> lock(m_);
                if (work_.empty()) return;
                f = std::move(work_.front());
                work_.pop_front();
            }
            f();
        }
    }
    size_t waiting() {
        std::lock_guard<std::mutex> lock(m_);
        return work_.size();
    }

private:
    std::mutex m_;
    std::deque<std::function<void()>> work_;
};
struct SimEvent {};
using hipStream_t = SimStream*;
using hipEvent_t = SimEvent*;
struct hipDeviceProp_t { char gcnArchName[32]; int multiProcessorCount; };

struct Sim {
    SimStream null_stream;
    hipError_t pending = hipSuccess;      // what hipGetLastError reports next
    hipError_t launch_status = hipSuccess;  // status of the next launches; a launch that fails enqueues nothing
    int device_syncs = 0, num_cus = 256;
    bool capturing = false;               // what every stream says of itself
    SimStream* of(hipStream_t s) { return s ? s : &null_stream; }
};
inline Sim sim;

template <class F>
inline void sim_run_grid(dim3 grid, dim3 block, F f) {
    gridDim = grid;
    blockDim = block;
    for (unsigned b = 0; b < grid.x; ++b)
        for (unsigned t = block.x; t-- > 0;) {  // thread 0 last: what it does behind a barrier follows the others' work
            blockIdx = dim3(b);
            threadIdx = dim3(t);
            f();
        }
}
template <class K, class... A>
inline void hipLaunchKernelGGL(K kernel, dim3 grid, dim3 block, size_t, hipStream_t s, A... args) {
    if (sim.launch_status != hipSuccess) {
        sim.pending = sim.launch_status;
        return;
    }
    sim.of(s)->push([=] { sim_run_grid(grid, block, [&] { kernel(args...); }); });
}
// the closure that runs kernel `f` with the values its arguments hold now (defined by the test, which knows the kernels)
std::function<void()> sim_bind(const void* f, void** args);
inline hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t s) {
    if (sim.launch_status != hipSuccess) return sim.pending = sim.launch_status;
    auto once = sim_bind(f, args);
    sim.of(s)->push([=] { sim_run_grid(grid, block, once); });
    return hipSuccess;
}
inline const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "simulated error"; }
inline hipError_t hipGetLastError() { hipError_t e = sim.pending; sim.pending = hipSuccess; return e; }
inline hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = sim.num_cus;
    return hipSuccess;
}
template <class T>
inline hipError_t hipMalloc(T** p, size_t n) { *p = static_cast<T*>(std::malloc(n)); return hipSuccess; }
inline hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
template <class T>
inline hipError_t hipHostMalloc(T** p, size_t n, unsigned) { *p = static_cast<T*>(std::malloc(n)); return hipSuccess; }
inline hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
inline hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
template <class T>
inline hipError_t hipGetSymbolAddress(void** p, T* symbol) { *p = symbol; return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = new SimStream; return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t s) { sim.of(s)->run(); return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = sim.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { ++sim.device_syncs; sim.null_stream.run(); return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { *e = new SimEvent; return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new SimEvent; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
