// A run of Algorithm 1 in one launch, for objectives and updates that are per-coordinate: an interaction reads and
// writes only its own coordinate of the two models, the initiator's snapshot and (with local steps inside) the
// initiator's objective data, so every tile of 256 or 512 coordinates can go through all interactions of the
// run on its own.  One workgroup per tile keeps the tile of all n models in local memory (1 or 2 KiB per node) from
// the first interaction to the last; its waves take the interactions in turn, in an order in which every interaction comes
// after the earlier ones that touch its nodes, and a wave waits for those by the number of interactions each of its two
// nodes has been through: the local steps for the last interaction that the initiator led, which made its snapshot, the rest
// for the last ones of both.  (Same arithmetic as interact_tile, same results bit for bit.)
// An interaction reads what is not in local memory -- a_i, c_i and, unless the initiator's last interaction was its
// own, the snapshot -- and writes the snapshot unless the next interaction of the node writes it again.  Where tiles are few
// (AHEAD), snapshots are held in local memory too, and the noise of the first four steps is drawn ahead of the wait.
// Bound by vector instructions (405 counted per interaction and 256 coordinates at H = 3) and, with few tiles, by the chain of
// dependent interactions.  On complete graphs with 8-bit codes, steps that waited for both nodes and steps that wait for the
// snapshot: 64 nodes x 2^20, H = 3, 256 interactions 784 and 759 us (1636 in 28 launches that moved 34 B per
// interaction-coordinate at 5.6 TB/s), 31 x 2 000 000, H = 5, 100 interactions 745 and 693; and with few tiles 8 x 8888, H = 3,
// 64 interactions 53.8, 42.2 and with AHEAD 33.6, 9 x 20 000, H = 3, 128 interactions 90.3, 71.1 and 53.4.
// The wait always ends: the waves of a workgroup are resident together, and the earliest interaction that is not
// finished waits for none.
#include <algorithm>

#include "diag_steps.hpp"
#include "interact_run.hpp"
#include "round_tile.hpp"

namespace swarm {

// The generator's words of an interaction: two per float4 of the lane, for the initiator's row and for the responder's.
// F = 2: a call per row, shared by a lane pair as everywhere (pair_words).  F = 1: a lane pair has one group of 8
// coordinates; the even lane calls for the initiator's row, the odd lane for the responder's, and the same exchange
// leaves each lane with its words of both.
template <int F>
struct RowWords { uint32_t i[F][2], j[F][2]; };
template <int F>
__device__ __forceinline__ RowWords<F> row_words(uint64_t seed, uint32_t ni, uint32_t nj, uint32_t event, uint64_t tile, uint32_t lane) {
    if constexpr (F == 2) {
        const LaneRandom wi = row_random(seed, ni, event, tile, lane), wj = row_random(seed, nj, event, tile, lane);
        return RowWords<F>{{{wi.a0, wi.a1}, {wi.b0, wi.b1}}, {{wj.a0, wj.a1}, {wj.b0, wj.b1}}};
    } else {
        const LaneRandom w = pair_words(stream(seed, TAG_SR, 0, (lane & 1u) ? nj : ni, event, tile * 32 + (lane >> 1)));
        return RowWords<F>{{{w.a0, w.a1}}, {{w.b0, w.b1}}};
    }
}

// What a run reads again: objective data and snapshots, of which all tiles under way together stay in cache.
__device__ __forceinline__ f4 ldg(const float *row, uint32_t off) { return *(SWARM_GLOBAL const f4 *)at_bytes(uniform(row), 4u * off); }
__device__ __forceinline__ void stg(float *row, uint32_t off, f4 v) { *(SWARM_GLOBAL f4 *)at_bytes(uniform(row), 4u * off) = v; }

// Gradient noise of steps q and q + 1 for a tile of 256 coordinates: the even lane of a pair draws for step q, the odd lane for
// step q + 1, and the exchange leaves each lane with its words of both steps.
__device__ __forceinline__ void two_noises(f4 &n0, f4 &n1, uint32_t q, uint32_t node, uint64_t tile, uint32_t lane, float scale,
                                           uint64_t seed, uint32_t event) {
    const LaneRandom r = pair_words(stream(seed, TAG_NOISE, q + (lane & 1u), node, event, tile * 32 + (lane >> 1)));
    float z0, z1, z2, z3;
    box_muller16(r.a0, scale, z0, z1);
    box_muller16(r.a1, scale, z2, z3);
    n0 = f4{z0, z1, z2, z3};
    box_muller16(r.b0, scale, z0, z1);
    box_muller16(r.b1, scale, z2, z3);
    n1 = f4{z0, z1, z2, z3};
}
__device__ __forceinline__ float noise_scale(float sigma) { return -1.3862943611198906f * sigma * sigma; }     // -2 ln 2 sigma^2

// Local steps q .. H - 1 of the lane's F float4 (diag_steps; F = 2: from the first).
template <bool NOISE, int F>
__device__ __forceinline__ void run_steps(f4 w[F], const f4 a[F], const f4 c[F], uint32_t node, uint64_t tile, uint32_t lane,
                                          uint32_t q, uint32_t H, float lr, float sigma, uint64_t seed, uint32_t event) {
    if constexpr (F == 2) {
        diag_steps<NOISE>(w[0], w[1], a[0], a[1], c[0], c[1], node, tile, lane, H, lr, sigma, seed, event);
    } else {
        for (; q < H; q += 2) {
            f4 n0 = {0.f, 0.f, 0.f, 0.f}, n1 = n0;
            if (NOISE) two_noises(n0, n1, q, node, tile, lane, noise_scale(sigma), seed, event);
            w[0] = diag_update(w[0], a[0], c[0], n0, lr);
            if (q + 1 < H) w[0] = diag_update(w[0], a[0], c[0], n1, lr);
        }
    }
}

// LOCAL: 0 = the pending update is W_i - Xhat_i where the descriptor says so; 1 / 2 = local steps of the diagonal
// objective in registers, with / without gradient noise.  RW: waves per workgroup.  F: float4 per lane, a tile has 256 F
// coordinates.
template <int BITS, int LOCAL, int RW, int F, bool AHEAD>
__global__ __launch_bounds__(RW * 64, F == 2 || AHEAD ? 4 : 7) void interact_run_kernel(const RunArgs ra) {
    constexpr uint32_t COORDS = 256 * F, ROW = 64 * F;           // of a tile: coordinates, float4
    constexpr int EARLY = AHEAD && LOCAL == 1 ? 4 : 0;           // steps whose noise is drawn ahead of the wait
    extern __shared__ f4 rows[];                  // n x COORDS floats; AHEAD: then the snapshots
    __shared__ uint32_t done[RUN_MAX_NODES];      // interactions each node has been through
    const GossipArgs &a = ra.g;
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t tile = blockIdx.x, base = tile * COORDS;
    bool in[F];
    uint32_t from[F], to[F];                      // coordinates of the tile: loaded from (past the row end: its last float4), stored to
#pragma unroll
    for (int f = 0; f < F; ++f) {
        to[f] = 4u * lane + 256u * f;
        in[f] = base + to[f] < a.d;
        from[f] = in[f] ? to[f] : (uint32_t)(a.d - 4 - base);
    }
    for (uint32_t u = threadIdx.x; u < a.n; u += RW * 64) done[u] = 0;
    constexpr int AT_ONCE = 8 / F;                // rows in flight per wave
    const uint32_t all = AHEAD ? 2 * a.n : a.n;
    auto row_of = [&](uint32_t u) { return u < a.n ? a.X + (uint64_t)u * a.d + base : a.Xhat + (uint64_t)(u - a.n) * a.d + base; };
    for (uint32_t u0 = wave; u0 < all; u0 += AT_ONCE * RW) {
        f4 v[AT_ONCE][F];
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const float *x = row_of(min(u0 + i * RW, all - 1));
#pragma unroll
            for (int f = 0; f < F; ++f) v[i][f] = ldg_nt(x, from[f]);
        }
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i)
            if (u0 + i * RW < all) {
#pragma unroll
                for (int f = 0; f < F; ++f) rows[(u0 + i * RW) * ROW + lane + 64 * f] = v[i][f];
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
    f4 oa[F] = {}, oc[F] = {};
    auto fetch_objective = [&](uint32_t node) {
        const uint64_t at = (uint64_t)node * a.d + base;
#pragma unroll
        for (int f = 0; f < F; ++f) { oa[f] = ldg(ra.A + at, from[f]); oc[f] = ldg(ra.C + at, from[f]); }
    };
    if (LOCAL && wave < ra.count) fetch_objective(next.nodes & 0xFFFFu);
    auto through = [&](uint32_t node) { return first_lane(__hip_atomic_load(&done[node], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)); };
    for (uint32_t k = wave; k < ra.count; k += RW) {
        const RunDesc rd = next;
        next = run_desc(ra.descs, k + RW, ra.count);
        const uint32_t event = rd.event, flags = rd.flags, turn = rd.turn, ni = rd.nodes & 0xFFFFu, nj = rd.nodes >> 16;
        const uint64_t at = (uint64_t)ni * a.d + base;
        RowWords<F> words{};
        if (BITS > 0) words = row_words<F>(a.seed, ni, nj, event, tile, lane);
        f4 *ri = rows + ni * ROW + lane, *rj = rows + nj * ROW + lane, *snap = ri + a.n * ROW;       // snap: AHEAD only
        float *hi = a.Xhat + at;
        f4 xi[F], xj[F], delta[F], average[F];
#pragma unroll
        for (int f = 0; f < F; ++f) delta[f] = zero;
        f4 early[EARLY + 1];
        if constexpr (EARLY > 0) {
            const uint32_t H = (flags >> 8) & 0xFFu;
#pragma unroll
            for (int q = 0; q < EARLY; q += 2)
                if ((uint32_t)q < H) two_noises(early[q], early[q + 1], q, ni, tile, lane, noise_scale(ra.sigma), a.seed, event);
        }
        if (LOCAL || (flags & SEQ_HAS_DELTA)) {
            while (through(ni) < flags >> RUN_READY_SHIFT) __builtin_amdgcn_s_sleep(1);       // the snapshot
            f4 h[F], w[F];
            if (AHEAD || (flags & RUN_SNAPSHOT_IS_MODEL)) {
#pragma unroll
                for (int f = 0; f < F; ++f) h[f] = (AHEAD ? snap : ri)[64 * f];
            } else {
#pragma unroll
                for (int f = 0; f < F; ++f) h[f] = ldg(hi, from[f]);
            }
#pragma unroll
            for (int f = 0; f < F; ++f) w[f] = h[f];
            if (LOCAL) {
                f4 a0[F], c0[F];
#pragma unroll
                for (int f = 0; f < F; ++f) { a0[f] = oa[f]; c0[f] = oc[f]; }
                if (k + RW < ra.count) fetch_objective(next.nodes & 0xFFFFu);
                const uint32_t H = (flags >> 8) & 0xFFu;
#pragma unroll
                for (int q = 0; q < EARLY; ++q)
                    if ((uint32_t)q < H) w[0] = diag_update(w[0], a0[0], c0[0], early[q], ra.lr);
                run_steps<LOCAL == 1, F>(w, a0, c0, ni, tile, lane, EARLY, H, ra.lr, ra.sigma, a.seed, event);
            } else {
#pragma unroll
                for (int f = 0; f < F; ++f) w[f] = ldg_nt(a.W + at, from[f]);
            }
#pragma unroll
            for (int f = 0; f < F; ++f) delta[f] = w[f] - h[f];
        }
        while ((through(ni) ^ (turn & 0xFFFFu)) | (through(nj) ^ (turn >> 16))) __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int f = 0; f < F; ++f) { xi[f] = ri[64 * f]; xj[f] = rj[64 * f]; }
        if constexpr (BITS > 0) {
            const float half_eps = 0.5f * a.eps;
            uint64_t codes_i[F], codes_j[F];
#pragma unroll
            for (int f = 0; f < F; ++f) {
                bool far = false;
                int missed = 0, zi[4], zj[4];
                codes_i[f] = round_float4<BITS>(xi[f], words.i[f][0], words.i[f][1], a.inv_eps, zi, far);
                codes_j[f] = round_float4<BITS>(xj[f], words.j[f][0], words.j[f][1], a.inv_eps, zj, far);
                average[f] = averaged<BITS>(zi, codes_j[f], xi[f], zero, a.inv_eps, half_eps, zj, missed, far);
                fails += in[f] ? missed : 0;
                clamped |= in[f] && far;
            }
            auto publish = [&](uint32_t node, const uint64_t codes[F]) {
                uint8_t *pub = a.ring + (uint64_t)node * a.row_bytes + base * BITS / 8;
#pragma unroll
                for (int f = 0; f < F; ++f)
                    if (in[f]) store_tile_code<BITS>(pub, to[f] / 4, codes[f]);
            };
            if (flags & RUN_LAST_OF_I) publish(ni, codes_i);      // the register keeps the code of the node's last interaction
            if (flags & RUN_LAST_OF_J) publish(nj, codes_j);
        } else {
#pragma unroll
            for (int f = 0; f < F; ++f) average[f] = 0.5f * (xi[f] + xj[f]);
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const f4 o = average[f] + delta[f];
            ri[64 * f] = o;
            rj[64 * f] = average[f];
            if (AHEAD) snap[64 * f] = o;
            else if (!(flags & RUN_SNAPSHOT_SHORT) && in[f]) stg(hi, to[f], o);
        }
        __hip_atomic_store(&done[ni], (turn & 0xFFFFu) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);   // every lane:
        __hip_atomic_store(&done[nj], (turn >> 16) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);       // no branch
    }
    if (BITS > 0) report(a.counters, fails, clamped);
    __syncthreads();
    for (uint32_t u = wave; u < a.n; u += RW)
        if (done[u] != 0) {
            float *x = a.X + (uint64_t)u * a.d + base;
#pragma unroll
            for (int f = 0; f < F; ++f)
                if (in[f]) stg_nt(x, to[f], rows[u * ROW + lane + 64 * f]);
            if constexpr (AHEAD) {
#pragma unroll
                for (int f = 0; f < F; ++f)
                    if (in[f]) stg_nt(a.Xhat + (uint64_t)u * a.d + base, to[f], rows[(a.n + u) * ROW + lane + 64 * f]);
            }
        }
}

template <int BITS, int LOCAL, int RW, int F, bool AHEAD = false>
static void launch_tiles(const RunArgs &ra, hipStream_t st) {
    const dim3 grid((unsigned)((ra.g.d + 256 * F - 1) / (256 * F)));
    interact_run_kernel<BITS, LOCAL, RW, F, AHEAD><<<grid, RW * 64, (size_t)ra.g.n * 256 * F * (AHEAD ? 2 : 1) * sizeof(float), st>>>(ra);
}

// Waves per workgroup, size of its tile and whether noise and snapshots are held ahead, by the number of nodes (how many
// interactions can run side by side, and how much local memory a tile takes) and of tiles.  512-coordinate tiles (F = 2) issue
// the fewest instructions, 256-coordinate ones leave room for more workgroups per compute unit and finish an interaction
// sooner.  With one or two workgroups per compute unit the chain of interactions is what takes the time, and a wave that has
// drawn its noise and finds the snapshot in local memory shortens it; with more, the waves that this leaves out are
// missed.  us per run, H = 3:  waves, F, A where ahead
//   d, interactions            4,1   8,1  12,1   2,2   4,2 |  4,1A  8,1A 12,1A 16,1A
//   n =  8,     8 888,  64      43    41    42    85    57 |    36    34    35    35
//            131 072, 128       89    91    96   158   104 |    77    75   110   112
//            262 144, 128      126   153   178   211   134 |   116   138   213   217
//          1 200 000, 128      428   586   769   484   446 |   431   586
//          2 400 000, 128      791  1114  1477   802   809 |   811  1120
//          3 200 000, 100      818  1156         793   824 |   834  1165
//   n = 16,   20 000, 200       94    73    73   236   129 |    82    63    62    62
//            131 072, 200      112   103   107   239   129 |   106    94   118   119
//            200 000, 200      169   173   195   327   176 |   168   171   228   231
//            400 000, 200      256   277   326   340   280 |   270   286   397   401
//          1 600 000, 100      410   482         639   415 |   443   505
//          4 000 000, 100     1002  1172  1436  1430   958 |  1063  1241
//   n = 31,   65 536, 200       92    61    58   241   125 |    84    60    56    54
//            131 072, 200      115    93    92   247   129 |   111    96   108   105
//   n = 64,   65 536, 256      121    79    68   319   163 |   110    80    73    70
// For 20 to 39 nodes 8 waves, F = 2 and 1: 32 x 500 000, 256 interactions: 349 and 357, 31 x 196 608, 128: 112 and 95.  The line between
// these two was not measured again since steps are taken ahead of the wait for both nodes.
struct TileForm { uint32_t waves, f; bool ahead; };
static TileForm tile_form(uint32_t n, uint64_t d) {
    constexpr uint64_t MANY = 5u << 19;           // coordinates
    if (n <= 9) return d <= 1u << 17 ? TileForm{8, 1, true} : d < 1u << 19 ? TileForm{4, 1, true} : d < MANY ? TileForm{4, 1, false} : TileForm{2, 2, false};
    if (n <= 19) return d <= 1u << 17 ? TileForm{8, 1, true} : d <= 3u << 16 ? TileForm{4, 1, true} : d < MANY ? TileForm{4, 1, false} : TileForm{4, 2, false};
    if (n <= 39) return d <= 1u << 16 ? TileForm{16, 1, true} : TileForm{8, d < 1u << 18 ? 1u : 2u, false};
    return {12, 1, false};
}

// Whether one launch is sooner done with m interactions that form so many dependency levels than a launch per level.
//  - It reads and writes every node's model once, whether or not the run touches it, and 12 to 16 B per
//    interaction-coordinate instead of 32 and two codes, so it needs enough interactions: 64 nodes x 2^20, H = 3, 8-bit
//    codes, 16 interactions 125 us with one launch per level, 135 in one launch; 24: 176 and 166; 32 nodes: 8 interactions
//    77 and 98, 12: 102 and 97.  Interactions that do not depend on one another at all (one level) have nothing to keep.
//  - Below 3 x 2^17 coordinates a level is all launch (5 us): one launch is sooner done whatever the graph (star of 64 nodes
//    x 200 000, H = 3, 64 interactions: 443 and 235 us; x 400 000: 459 and 424; of 78 x 100 000, H = 20: 1128 and 358).
//  - Above, only as many waves of a compute unit work as it has workgroups times interactions side by side; a level keeps
//    them all busy.  In units of 256 coordinates that have to be 5 up to three local steps and 1.4 per step beyond (14
//    suffice).  By levels and in one launch, hubs joined to all other nodes, about as many interactions as nodes:
//      24 x 4 000 000, H = 10, 1 hub   750  1600    4 hubs  661  765    40 x 2^20, H = 3, 2 hubs   273  383    4 hubs  298  269
//      48 x 4 000 000, H = 5, 1 hub   1364  3087    3 hubs 1225 1499    64 x 4 000 000, H = 20, 4 hubs  2631  3273
//      31 x 2^20, H = 5, 1 hub         292   382    3 hubs  243  217    19 x 4 000 000, H = 20, 1 hub    883   971
//    Complete graphs, rings and paths are wide enough up to H = 5 (64 x 4 000 000, H = 20, path, 64 interactions: 2611, 2273).
bool interact_run_pays(uint64_t d, uint32_t n, uint32_t H, uint32_t m, uint32_t levels) {
    if (n > RUN_MAX_NODES || levels <= 1 || 8 * (uint64_t)m < 3 * (uint64_t)n) return false;
    if (d < 3u << 17) return true;
    // waves and tiles as they were when the line was drawn, with steps that waited for both nodes
    const TileForm form = n <= 9 && d >= 1u << 19 ? TileForm{2, 2, false} : n <= 19 ? TileForm{4, 1, false} : tile_form(n, d);
    const uint32_t by_memory = 160u / (n * form.f + 1), by_waves = (form.f == 2 ? 16u : 28u) / form.waves;
    const double side_by_side = std::min((double)m / levels, (double)form.waves);
    const double need = std::min(std::max(1.4 * H, 5.0), 14.0);
    return form.f * std::min(by_memory, by_waves) * side_by_side >= need;
}

template <int BITS, int LOCAL>
static void launch_waves(const RunArgs &ra, hipStream_t st) {
    const TileForm form = tile_form(ra.g.n, ra.g.d);
    if (form.ahead) {
        if (form.waves == 4) launch_tiles<BITS, LOCAL, 4, 1, true>(ra, st);
        else if (form.waves == 8) launch_tiles<BITS, LOCAL, 8, 1, true>(ra, st);
        else launch_tiles<BITS, LOCAL, 16, 1, true>(ra, st);
    } else if (form.waves == 2) launch_tiles<BITS, LOCAL, 2, 2>(ra, st);
    else if (form.waves == 4 && form.f == 2) launch_tiles<BITS, LOCAL, 4, 2>(ra, st);
    else if (form.waves == 4) launch_tiles<BITS, LOCAL, 4, 1>(ra, st);
    else if (form.waves == 12) launch_tiles<BITS, LOCAL, 12, 1>(ra, st);
    else if (form.f == 2) launch_tiles<BITS, LOCAL, 8, 2>(ra, st);
    else launch_tiles<BITS, LOCAL, 8, 1>(ra, st);
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
