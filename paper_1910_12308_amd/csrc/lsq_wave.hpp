// Sums over a wave of several values per lane, and its largest value (least-squares and softmax kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swarm {

// What the lane S away holds, without a turn through local memory (S up to 8: inside a row of 16 lanes).
template <int S>
__device__ __forceinline__ float across(float x) {
    const int i = (int)__float_as_uint(x);
    int r;
    if constexpr (S == 1) r = __builtin_amdgcn_mov_dpp(i, 0xB1, 0xF, 0xF, true);             // quad [1, 0, 3, 2]
    else if constexpr (S == 2) r = __builtin_amdgcn_mov_dpp(i, 0x4E, 0xF, 0xF, true);        // quad [2, 3, 0, 1]
    else if constexpr (S == 4)                                                               // half a row mirrored, then its quads
        r = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(i, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else r = __builtin_amdgcn_mov_dpp(i, 0x128, 0xF, 0xF, true);                             // a row turned by 8
    static_assert(S == 1 || S == 2 || S == 4 || S == 8, "");
    return __uint_as_float((uint32_t)r);
}
// The sum of a lane's value and that of the lane S away: of `low` in lanes whose bit S is clear, of `high` in the others.
template <int S>
__device__ __forceinline__ float paired(float low, float high, uint32_t lane) {
    if constexpr (S >= 16) {
        const uint32_t l = __float_as_uint(low), h = __float_as_uint(high);
        if constexpr (S == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(l, h, false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(l, h, false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
    } else {
        const float keep = (lane & S) ? high : low, give = (lane & S) ? low : high;
        return keep + across<S>(give);
    }
}

// The wave's sums of R per-lane values, by halving: a lane gives half of its values to the lane a power of two
// away and keeps the other half, so that about R exchanges (not 6 R) leave the total of value `(lane * R / (2 * TOP)) % R` in
// the lane.  TOP: the first distance; the order of a value's sum is by distances TOP, TOP / 2 .. 1, 2 TOP .. 32.
template <int N, int S>
__device__ __forceinline__ void halve(float *v, uint32_t lane) {
    if constexpr (N >= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = paired<S>(v[i], v[i + N], lane);
    } else {
        v[0] = paired<S>(v[0], v[0], lane);
    }
    if constexpr (S > 1) halve<N / 2, S / 2>(v, lane);
}
template <int S>
__device__ __forceinline__ float total_from(float t, uint32_t lane) {       // over distances S .. 32
    if constexpr (S >= 64) return t;
    else return total_from<2 * S>(paired<S>(t, t, lane), lane);
}
template <int R, int TOP = R / 2>
__device__ __forceinline__ float wave_totals(float v[R], uint32_t lane) {
    halve<R / 2, TOP>(v, lane);
    return total_from<2 * TOP>(v[0], lane);
}

// The largest value of the wave, in every lane.
template <int S = 32>
__device__ __forceinline__ float wave_maximum(float x) {
    if constexpr (S == 0) return x;
    else if constexpr (S >= 16) {
        const uint32_t u = __float_as_uint(x);
        const auto r = S == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return wave_maximum<S / 2>(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
    } else return wave_maximum<S / 2>(fmaxf(x, across<S>(x)));
}

}  // namespace swarm
