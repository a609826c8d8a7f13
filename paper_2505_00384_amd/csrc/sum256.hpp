// Fixed-order workgroup sum shared by the kernels that reduce the same
// partial sums independently (every workgroup of a launch, or two different
// kernels, obtain the same bits).
#pragma once

#include <hip/hip_runtime.h>

namespace hx {

// Sum of p[0..nb) by the first 256 threads of a workgroup of at least 256
// (every thread calls it): thread t < 256 adds p[t], p[t + 256], ...
// starting from 0; each wave folds its lanes with shuffle-down distances 32,
// 16, ..., 1; the four wave sums are added in wave order starting from 0.
// Every thread returns the result.  The host function host_sum256
// (solver.cpp) performs the same additions in the same order.
__device__ inline double sum256(const double *__restrict__ p, int nb, double *sh /* LDS [4] */)
{
    double s = 0.0;
    if (threadIdx.x < 256) {
        // eight loads in flight at a time; the additions in the same order
        // (an element past the end adds zero)
        for (int i0 = threadIdx.x; i0 < nb; i0 += 8 * 256) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = i0 + 256 * u < nb ? p[i0 + 256 * u] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0 && wv < 4) sh[wv] = s;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) t += sh[q];
    __syncthreads();
    return t;
}

// A value the host reads after an event on the stream (pinned, device-mapped
// memory): a system-scope store, and host_stores_done() in the same wave
// afterwards waits until its stores have arrived, so the wave, and with it
// the kernel that the event follows, does not end before.
__device__ __forceinline__ void host_store(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void host_stores_done() { __builtin_amdgcn_s_waitcnt(0); }

}  // namespace hx
