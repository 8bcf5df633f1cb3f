// Sums over a wave of several values per lane (least-squares kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swarm {

// The wave's sums of R per-lane values, by halving: a lane gives half of its values to the lane a power of two
// away and keeps the other half, so that about R exchanges (not 6 R) leave the total of value `lane % R` in the lane.
template <int N, int R>
__device__ __forceinline__ void halve(float v[R], uint32_t lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float keep = (lane & N) ? v[i + N] : v[i], give = (lane & N) ? v[i] : v[i + N];
        v[i] = keep + __shfl_xor(give, N);
    }
    if constexpr (N > 1) halve<N / 2, R>(v, lane);
}
template <int R>
__device__ __forceinline__ float wave_totals(float v[R], uint32_t lane) {
    halve<R / 2, R>(v, lane);
    float t = v[0];
#pragma unroll
    for (int off = R; off < 64; off *= 2) t += __shfl_xor(t, off);
    return t;
}

}  // namespace swarm
