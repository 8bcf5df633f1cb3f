// A run of Algorithm 1 in one launch, for objectives and updates that are per-coordinate: an interaction reads and
// writes only its own coordinate of the two models, the initiator's snapshot and (with local steps inside) the
// initiator's objective data, so every 512-coordinate tile of the matrix can go through all interactions of the
// run on its own.  One workgroup per tile keeps the tile of all n models in local memory (2 KiB per node) from the
// first interaction to the last; its waves take the interactions in turn, in an order in which every interaction comes
// after the earlier ones that touch its nodes, and a wave waits for those by the number of interactions each of its two
// nodes has been through.  (Same arithmetic as interact_tile, same results bit for bit.)
// An interaction reads what is not in local memory -- a_i, c_i and, unless the initiator's last interaction was its
// own, the snapshot -- and writes the snapshot unless the next interaction of the node writes it again.
// Bound by vector instructions (about 520 per interaction and tile at H = 3) and by how many interactions can run side
// by side: 64 nodes x 2^20, H = 3, 8-bit codes, 256 interactions on a complete graph take 920 us, against 1636 us for 28
// launches that moved 34 B per interaction-coordinate at 5.6 TB/s; 16 nodes x 300 000, 200 interactions 353 us
// against 1511; 8 nodes x 8888, 64 interactions 79 us against 249.  (Without the requests ahead of the wait and the
// skipped snapshots: 1046 us.)
// The wait always ends: the waves of a workgroup are resident together, and the earliest interaction that is not
// finished waits for none.
#include "diag_steps.hpp"
#include "interact_run.hpp"
#include "round_tile.hpp"

namespace swarm {

// LOCAL: 0 = the pending update is W_i - Xhat_i where the descriptor says so; 1 / 2 = local steps of the diagonal
// objective in registers, with / without gradient noise.  RW: waves per workgroup.
template <int BITS, int LOCAL, int RW>
__global__ __launch_bounds__(RW * 64, 4) void interact_run_kernel(const RunArgs ra) {
    extern __shared__ f4 rows[];                  // n x TILE floats
    __shared__ uint32_t done[RUN_MAX_NODES];      // interactions each node has been through
    const GossipArgs &a = ra.g;
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t tile = blockIdx.x;
    const TilePos t = tile_pos<false>(tile, lane, a.d);
    static_assert(RW * 64 >= RUN_MAX_NODES, "one thread per node");
    if (threadIdx.x < a.n) done[threadIdx.x] = 0;
    for (uint32_t u0 = wave; u0 < a.n; u0 += 4 * RW) {          // four rows in flight per wave
        f4 v[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float *x = a.X + (uint64_t)min(u0 + i * RW, a.n - 1) * a.d + t.base;
            v[i][0] = ldg_nt(x, t.oA);
            v[i][1] = ldg_nt(x, t.oB);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (u0 + i * RW < a.n) {
                rows[(u0 + i * RW) * (TILE / 4) + lane] = v[i][0];
                rows[(u0 + i * RW) * (TILE / 4) + lane + 64] = v[i][1];
            }
    }
    __syncthreads();
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    bool clamped = false;
    int fails = 0;
    // Interactions k = wave, wave + RW, ...: no branch of this loop depends on the lane except around global stores, so
    // the wave stays together whatever the compiler makes of it.  What does not depend on the interactions before --
    // the next descriptor, its objective data, the random words -- is requested or computed ahead of the wait.
    RunDesc next = run_desc(ra.descs, wave, ra.count);
    f4 aA = zero, aB = zero, cA = zero, cB = zero;
    auto fetch_objective = [&](uint32_t node) {
        const uint64_t at = (uint64_t)node * a.d + t.base;
        aA = ldg_nt(ra.A + at, t.oA); aB = ldg_nt(ra.A + at, t.oB);
        cA = ldg_nt(ra.C + at, t.oA); cB = ldg_nt(ra.C + at, t.oB);
    };
    if (LOCAL && wave < ra.count) fetch_objective(next.nodes & 0xFFFFu);
    for (uint32_t k = wave; k < ra.count; k += RW) {
        const RunDesc rd = next;
        next = run_desc(ra.descs, k + RW, ra.count);
        const uint32_t event = rd.event, flags = rd.flags, turn = rd.turn, ni = rd.nodes & 0xFFFFu, nj = rd.nodes >> 16;
        const uint64_t at = (uint64_t)ni * a.d + t.base;
        LaneRandom ni_words{}, nj_words{};
        if (BITS > 0) {
            ni_words = row_random(a.seed, ni, event, tile, lane);
            nj_words = row_random(a.seed, nj, event, tile, lane);
        }
        while ((first_lane(__hip_atomic_load(&done[ni], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) ^ (turn & 0xFFFFu)) |
               (first_lane(__hip_atomic_load(&done[nj], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) ^ (turn >> 16)))
            __builtin_amdgcn_s_sleep(1);
        f4 *ri = rows + ni * (TILE / 4) + lane, *rj = rows + nj * (TILE / 4) + lane;
        float *hi = a.Xhat + at;
        const f4 xiA = ri[0], xiB = ri[64], xjA = rj[0], xjB = rj[64];
        f4 dA = zero, dB = zero;
        if (LOCAL || (flags & SEQ_HAS_DELTA)) {
            f4 hA = xiA, hB = xiB;
            if (!(flags & RUN_SNAPSHOT_IS_MODEL)) { hA = ldg_nt(hi, t.oA); hB = ldg_nt(hi, t.oB); }
            f4 wA = hA, wB = hB;
            if (LOCAL) {
                const f4 a0 = aA, a1 = aB, c0 = cA, c1 = cB;
                if (k + RW < ra.count) fetch_objective(next.nodes & 0xFFFFu);
                diag_steps<LOCAL == 1>(wA, wB, a0, a1, c0, c1, ni, tile, lane, (flags >> 8) & 0xFFu, ra.lr, ra.sigma, a.seed, event);
            } else {
                const float *wi = a.W + at;
                wA = ldg_nt(wi, t.oA); wB = ldg_nt(wi, t.oB);
            }
            dA = wA - hA;
            dB = wB - hB;
        }
        f4 avgA, avgB;
        if constexpr (BITS > 0) {
            bool clampedA = false, clampedB = false;
            int failsA = 0, failsB = 0;
            int ziA[4], ziB[4], zjA[4], zjB[4];
            const uint64_t ciA = round_float4<BITS>(xiA, ni_words.a0, ni_words.a1, a.inv_eps, ziA, clampedA);
            const uint64_t ciB = round_float4<BITS>(xiB, ni_words.b0, ni_words.b1, a.inv_eps, ziB, clampedB);
            const uint64_t cjA = round_float4<BITS>(xjA, nj_words.a0, nj_words.a1, a.inv_eps, zjA, clampedA);
            const uint64_t cjB = round_float4<BITS>(xjB, nj_words.b0, nj_words.b1, a.inv_eps, zjB, clampedB);
            const float half_eps = 0.5f * a.eps;
            avgA = averaged<BITS>(ziA, cjA, xiA, zero, a.inv_eps, half_eps, zjA, failsA, clampedA);
            avgB = averaged<BITS>(ziB, cjB, xiB, zero, a.inv_eps, half_eps, zjB, failsB, clampedB);
            if (flags & RUN_LAST_OF_I) {          // the register keeps the code of the node's last interaction
                uint8_t *pub = ring_tile<BITS>(a, 0, ni, t);
                if (t.inA) store_tile_code<BITS>(pub, t.cA / 4, ciA);
                if (t.inB) store_tile_code<BITS>(pub, t.cB / 4, ciB);
            }
            if (flags & RUN_LAST_OF_J) {
                uint8_t *pub = ring_tile<BITS>(a, 0, nj, t);
                if (t.inA) store_tile_code<BITS>(pub, t.cA / 4, cjA);
                if (t.inB) store_tile_code<BITS>(pub, t.cB / 4, cjB);
            }
            fails += (t.inA ? failsA : 0) + (t.inB ? failsB : 0);
            clamped |= (t.inA && clampedA) || (t.inB && clampedB);
        } else {
            avgA = 0.5f * (xiA + xjA);
            avgB = 0.5f * (xiB + xjB);
        }
        const f4 oA = avgA + dA, oB = avgB + dB;
        ri[0] = oA; ri[64] = oB;
        rj[0] = avgA; rj[64] = avgB;
        if (!(flags & RUN_SNAPSHOT_SHORT)) {
            if (t.inA) stg_nt(hi, t.cA, oA);
            if (t.inB) stg_nt(hi, t.cB, oB);
        }
        __hip_atomic_store(&done[ni], (turn & 0xFFFFu) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);   // every lane:
        __hip_atomic_store(&done[nj], (turn >> 16) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);       // no branch
    }
    if (BITS > 0) report(a.counters, fails, clamped);
    __syncthreads();
    for (uint32_t u = wave; u < a.n; u += RW)
        if (done[u] != 0) {
            float *x = a.X + (uint64_t)u * a.d + t.base;
            const f4 xA = rows[u * (TILE / 4) + lane], xB = rows[u * (TILE / 4) + lane + 64];
            if (t.inA) stg_nt(x, t.cA, xA);
            if (t.inB) stg_nt(x, t.cB, xB);
        }
}

template <int BITS, int LOCAL>
static void launch_waves(const RunArgs &ra, hipStream_t st) {
    const dim3 grid((unsigned)((ra.g.d + TILE - 1) / TILE));
    const size_t lds = (size_t)ra.g.n * TILE * sizeof(float);
    // as many waves as a compute unit holds at this register count, shared by the workgroups that its local memory holds
    if (ra.g.n <= 19) interact_run_kernel<BITS, LOCAL, 4><<<grid, 4 * 64, lds, st>>>(ra);
    else if (ra.g.n <= 39) interact_run_kernel<BITS, LOCAL, 8><<<grid, 8 * 64, lds, st>>>(ra);
    else interact_run_kernel<BITS, LOCAL, 16><<<grid, 16 * 64, lds, st>>>(ra);
}

template <int BITS>
static void launch_form(const RunArgs &ra, int local, hipStream_t st) {
    if (local == 0) launch_waves<BITS, 0>(ra, st);
    else if (local == 1) launch_waves<BITS, 1>(ra, st);
    else launch_waves<BITS, 2>(ra, st);
}

hipError_t launch_interact_run(const GossipArgs &g, uint32_t bits, const RunDesc *descs_dev, uint32_t count,
                               const DiagObjective *local, float lr, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (g.n > RUN_MAX_NODES) return hipErrorInvalidValue;
    const RunArgs ra{g, descs_dev, count, local ? local->a : nullptr, local ? local->c : nullptr, local ? local->sigma : 0.f, lr};
    const int form = !local ? 0 : (local->sigma != 0.f ? 1 : 2);
    switch (bits) {
        case 0: launch_form<0>(ra, form, st); break;
        case 2: launch_form<2>(ra, form, st); break;
        case 4: launch_form<4>(ra, form, st); break;
        case 8: launch_form<8>(ra, form, st); break;
        case 16: launch_form<16>(ra, form, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace swarm
