// Whole round in one pass for per-coordinate objectives (diagonal quadratics): the H local steps of the
// matched nodes are taken in registers and fed straight into the quantized gossip step, so the live copy
// W never travels through memory.  Same arithmetic, in the same order, as local_diag_kernel followed by
// the gossip pass (the tile code is the shared one of round_tile.hpp with the steps as the source of the
// pending update); per pair-coordinate it reads X_i, X_j, a_i, a_j, c_i, c_j (24 B) and the two partner
// codes, and writes X_i', X_j' (8 B) and the two published codes.
#include "round_tile.hpp"

namespace swarm {

template <int BITS, int STALE, bool INPLACE, bool NOISE>
__global__ __launch_bounds__(WAVES * 64) void fused_pairs_kernel(const RoundArgs ra) {
    round_pairs_body<BITS, NOISE ? SRC_STEPS_NOISY : SRC_STEPS, STALE, INPLACE>(ra);
}

// Both reads of a pair are stale: one grid row per node (see round_node_tile).
// PER_SIMD: waves per SIMD the kernel is scheduled for, 0 = the compiler's choice (7 or 8).  See five_waves.
template <int BITS, bool INPLACE, bool NOISE, int PER_SIMD>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(PER_SIMD ? PER_SIMD : 1, PER_SIMD ? PER_SIMD : 8)))
void fused_nodes_kernel(const RoundArgs ra) {
    round_nodes_body<BITS, NOISE ? SRC_STEPS_NOISY : SRC_STEPS, INPLACE>(ra);
}

// Unmatched nodes: take the local steps and adopt the result; publish the code of the model that a
// partner would have read (the pre-step model when the apply is deferred).
template <int BITS, bool INPLACE, bool NOISE>
__global__ __launch_bounds__(WAVES * 64) void fused_singles_kernel(const RoundArgs ra) {
    round_singles_body<BITS, NOISE ? SRC_STEPS_NOISY : SRC_STEPS, INPLACE>(ra);
}

// Waves per SIMD of the rounds with codes of 2, 4 and 8 bits and both reads stale.  Bound by memory up to three noisy steps,
// by vector instructions beyond.  Left to itself the compiler takes 68 registers, seven waves and one Box-Muller chain
// after the other; with a step of 104 instead of 121 vector instructions that made the rounds bound by memory 1 to 3 %
// slower.  For six waves and fewer it puts the four chains of a step side by side (73 registers).  Five waves then stream
// best, and hide too little where a launch is short or the steps are many.  us (121 instructions, 7 waves; 104, 7;
// 104, 6; 104, 5), 64 nodes, 4 bits unless said:
//   25 600 000, H = 3           4512  4559  4513  4413     1 048 576, H = 5   219  202  200  205
//   4 000 000, H = 3             721   744   726   698     100 000, H = 3    30.5  29.9  30.0  31.1
//   12 000 000, 2 bits, H = 3   2121  2187  2151  2051     300 000, H = 3    66.3  65.9  66.0  65.8
//   4 000 000, H = 5             816   757   752   759     1 048 576, H = 1   190   190   190   187
// With 8 bits the compiler's choice and five, the best of four interleaved runs: 1 to 5 %; six are between them, and from four
// steps on or in shorter launches the choice is as good or better (16 nodes, 1 000 000, H = 4: 56.2, five 59.5).  With 16
// bits five and six gain nothing anywhere.
//   16 000 000, H = 2           3097  3069     1 048 576, H = 2           204  202     9 nodes, 16 000 000, H = 2   434  423
//   4 000 000, H = 3             779   739     1 048 576, H = 3           204  200     31 nodes, 1 000 000, H = 3   104  103
static bool five_waves(uint32_t H, uint64_t tiles) { return H <= 3 && tiles >= 1u << 15; }

template <int BITS, bool INPLACE, bool NOISE>
static void launch_nodes(const RoundArgs &ra, uint32_t H, dim3 grid, hipStream_t st) {
    constexpr int FEW = BITS == 8 ? 0 : 6;        // where there are not five
    if constexpr (BITS > 8) {
        fused_nodes_kernel<BITS, INPLACE, NOISE, 0><<<grid, WAVES * 64, 0, st>>>(ra);
    } else {
        if (five_waves(H, (uint64_t)grid.x * WAVES * grid.y))
            fused_nodes_kernel<BITS, INPLACE, NOISE, 5><<<grid, WAVES * 64, 0, st>>>(ra);
        else
            fused_nodes_kernel<BITS, INPLACE, NOISE, FEW><<<grid, WAVES * 64, 0, st>>>(ra);
    }
}

template <int BITS, bool INPLACE, bool NOISE>
static void launch_pairs_stale(const RoundArgs &ra, uint32_t H, int stale_mode, dim3 grid, hipStream_t st) {
    switch (stale_mode) {
        case 0: fused_pairs_kernel<BITS, 0, INPLACE, NOISE><<<grid, WAVES * 64, 0, st>>>(ra); break;
        case 1: launch_nodes<BITS, INPLACE, NOISE>(ra, H, dim3(grid.x, 2 * grid.y, 1), st); break;   // one grid row per node
        case 3: fused_pairs_kernel<BITS, 3, INPLACE, NOISE><<<grid, WAVES * 64, 0, st>>>(ra); break;
        default: fused_pairs_kernel<BITS, 2, INPLACE, NOISE><<<grid, WAVES * 64, 0, st>>>(ra); break;
    }
}

template <int BITS>
static void launch_bits(const RoundArgs &ra, bool inplace, bool noise, uint32_t H, int stale_mode, uint32_t npairs,
                        uint32_t nsingles, bool singles, hipStream_t st) {
    if (!singles) {
        const dim3 grid = tile_grid(ra.g.d, npairs);
        if (inplace) { if (noise) launch_pairs_stale<BITS, true, true>(ra, H, stale_mode, grid, st); else launch_pairs_stale<BITS, true, false>(ra, H, stale_mode, grid, st); }
        else { if (noise) launch_pairs_stale<BITS, false, true>(ra, H, stale_mode, grid, st); else launch_pairs_stale<BITS, false, false>(ra, H, stale_mode, grid, st); }
    } else {
        const dim3 grid = tile_grid(ra.g.d, nsingles);
        if (inplace) { if (noise) fused_singles_kernel<BITS, true, true><<<grid, WAVES * 64, 0, st>>>(ra); else fused_singles_kernel<BITS, true, false><<<grid, WAVES * 64, 0, st>>>(ra); }
        else { if (noise) fused_singles_kernel<BITS, false, true><<<grid, WAVES * 64, 0, st>>>(ra); else fused_singles_kernel<BITS, false, false><<<grid, WAVES * 64, 0, st>>>(ra); }
    }
}

static hipError_t dispatch(const GossipArgs &g, const DiagObjective &o, uint32_t bits, bool inplace, uint32_t H, float lr,
                           int stale_mode, uint32_t npairs, uint32_t nsingles, bool singles, hipStream_t st) {
    const RoundArgs ra{g, o.a, o.c, o.sigma, lr};
    const bool noise = o.sigma != 0.f;
    switch (bits) {
        case 2: launch_bits<2>(ra, inplace, noise, H, stale_mode, npairs, nsingles, singles, st); break;
        case 4: launch_bits<4>(ra, inplace, noise, H, stale_mode, npairs, nsingles, singles, st); break;
        case 8: launch_bits<8>(ra, inplace, noise, H, stale_mode, npairs, nsingles, singles, st); break;
        case 16: launch_bits<16>(ra, inplace, noise, H, stale_mode, npairs, nsingles, singles, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fused_pairs(const GossipArgs &g, const DiagObjective &o, uint32_t bits, bool inplace, uint32_t H,
                              float lr, int stale_mode, uint32_t npairs, hipStream_t st) {
    if (npairs == 0) return hipSuccess;
    return dispatch(g, o, bits, inplace, H, lr, stale_mode, npairs, 0, false, st);
}

hipError_t launch_fused_singles(const GossipArgs &g, const DiagObjective &o, uint32_t bits, bool inplace, uint32_t H,
                                float lr, uint32_t nsingles, hipStream_t st) {
    if (nsingles == 0) return hipSuccess;
    return dispatch(g, o, bits, inplace, H, lr, 0, 0, nsingles, true, st);
}

}  // namespace swarm
