// Device helpers shared by the HIP kernels of the gradient library (gfx950).
//
// Nothing here is shared with the CPU oracle: this is the GPU path only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pg {

constexpr int kWave = 64;  // CDNA wavefront width

// psi(s) = s^2/2 + log(1+s^2)/2 evaluated from q = s^2 (log1p keeps the
// small-|s| terms accurate).
__device__ __forceinline__ double psi_from_sq(double s2) { return 0.5 * s2 + 0.5 * log1p(s2); }

// psi'(s) = s + s/(1+s^2).
__device__ __forceinline__ double dpsi_from(double s, double s2) { return s + s / (1.0 + s2); }

// psi''(s) = 1 + (1-s^2)/(1+s^2)^2.
__device__ __forceinline__ double ddpsi_from_sq(double s2) {
    double q = 1.0 + s2;
    return 1.0 + (1.0 - s2) / (q * q);
}

// Sum over the 64 lanes of a wavefront; every lane receives the total.
// The butterfly order is fixed, so the result is bitwise repeatable.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Sum over a workgroup of BS threads (BS a multiple of 64, <= 1024); the
// total is valid in thread 0.  lds must hold BS/64 doubles.  Fixed order.
template <int BS>
__device__ __forceinline__ double block_sum(double v, double* lds) {
    constexpr int NW = BS / kWave;
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    if (NW == 1) return v;
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    double r = 0.0;
    if (wid == 0) {
        r = lane < NW ? lds[lane] : 0.0;
        r = wave_sum(r);
    }
    __syncthreads();
    return r;
}

// Runtime-size variant (blockDim.x a multiple of 64).
__device__ __forceinline__ double block_sum_dyn(double v, double* lds) {
    const int nw = blockDim.x / kWave;
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    if (nw == 1) return v;
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    double r = 0.0;
    if (wid == 0) {
        r = lane < nw ? lds[lane] : 0.0;
        r = wave_sum(r);
    }
    __syncthreads();
    return r;
}

// Workgroups of one launch are dealt round-robin to the 8 XCDs (each with its
// own L2).  Remap the hardware block id so that XCD x works on one contiguous
// range of logical blocks: neighbouring elements then share an L2, which is
// where the node values they gather (and the gradient lines they update) live.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nblocks) {
    constexpr uint32_t NX = 8;
    const uint32_t q = nblocks / NX, r = nblocks % NX;
    const uint32_t x = b % NX, i = b / NX;
    return x * q + (x < r ? x : r) + i;
}

// FP64 atomic add without return value: a hardware global_atomic_add_f64.
__device__ __forceinline__ void atomic_add_f64(double* p, double v) {
    unsafeAtomicAdd(p, v);
}

// Handing values to whichever workgroup finishes last, without device-scope
// fences.  A release fence writes back the whole L2 and an acquire fence
// invalidates it, some microseconds on a launch of a few; nothing else in
// those caches has to be seen.  So the values themselves go through the
// coherence point: a value is stored by an agent-scope atomic store (or added
// by an agent-scope atomic), the storing wave waits until its memory
// operations are performed (publish_wait), and only then is the ticket taken;
// the workgroup that finds itself last reads the values with agent-scope
// atomic loads, which never return a line an XCD's own cache still holds.
// Where several waves publish, each waits for its own before the workgroup
// barrier that precedes the ticket.
__device__ __forceinline__ void publish(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_wait() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the compiler keeps the order too
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
__device__ __forceinline__ double read_published(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Sum of p[0 .. n) by a workgroup of any size (whole waves), valid in thread
// 0, with the same bits whatever the size: as 1,024 threads would, entry t,
// t + 1024, ... to thread t, a butterfly per 64 of them, a butterfly over
// those 16.  lds holds 16 doubles.  PUB: the entries were published.
template <bool PUB>
__device__ __forceinline__ double final_sum_block(const double* __restrict__ p, int64_t n, double* lds) {
    constexpr int kU = 8, kVW = 16, kStride = kVW * kWave;  // loads in flight; virtual waves
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave, nw = blockDim.x / kWave;
    for (int vw = wid; vw < kVW; vw += nw) {
        double s = 0.0;
        for (int64_t q = vw * kWave + lane; q < n; q += kU * kStride) {
            double v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t i = q + u * kStride;
                v[u] = i < n ? (PUB ? __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                    : p[i])
                             : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (q + u * kStride < n) s += v[u];
        }
        s = wave_sum(s);
        if (lane == 0) lds[vw] = s;
    }
    __syncthreads();
    double r = 0.0;
    if (wid == 0) r = wave_sum(lane < kVW ? lds[lane] : 0.0);
    return r;
}

// Takes the ticket; true for the last of n, which leaves it at zero for the next
// launch.  The count wraps by itself: launches of n that overlap by mistake may
// mix up their sums, but n tickets each later it is at zero again (reset by the
// last one's store, it kept what others took in between, and no later launch
// of the plan found its last workgroup right).
__device__ __forceinline__ bool take_ticket(int32_t* ticket, int n) {
    return atomicInc(reinterpret_cast<unsigned*>(ticket), (unsigned)n - 1) == (unsigned)n - 1;
}

template <typename T>
__device__ __forceinline__ double to_f64(T v) {
    return static_cast<double>(v);
}

}  // namespace pg
