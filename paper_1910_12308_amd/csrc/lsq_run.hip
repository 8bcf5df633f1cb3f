// Algorithm 1 on small least-squares swarms: a run of interactions (or a single one) in one launch.  A workgroup owns
// 128 columns of all n models and snapshots and keeps them in local memory (1 KiB per node); each of its four waves
// takes every fourth interaction, in an order in which every interaction follows those it depends on, and waits in
// local memory for the earlier interactions of its two nodes (as in interact_run.hip).  A lane holds two columns: the
// batch's rows of A, the products with them and the update need no other lane but for the residuals, and of those only
// the sums over a workgroup's columns leave it.  The waves that run the same interaction in the other workgroups wait
// for these words in device memory, each tagged with the number of its step, so that nothing has to be cleared between
// steps; two sets of words alternate, because a wave writes its words of step c + 2 after it has read all words of step
// c + 1, and those were written by waves that had read step c.  Rows of the next step are requested before the wait.
// Bound by latency: a step is a chain of products, sums over the wave, one exchange through device memory (about half of
// its 2.5 us) and an update, two to four interactions run side by side.  8 nodes x 4096, batch 32, H = 2, 200
// interactions: 0.98 ms, against 1.75 ms for 112 launches of one interaction per 8 workgroups and row; a single
// interaction 12.6 us against 43.5 in two launches and a copy.  All workgroups on one die: no faster (1.01 ms).
// Four waves per workgroup are room for four interactions side by side: graphs that let many more run at once keep a launch
// per level (LSQ_RUN_WIDTH in swarm_api.hip).
// All workgroups are resident together (at most 64), the earliest unfinished interaction waits for none, and every
// wait is bounded, so that all waves end whatever happens to the others.
#include <type_traits>

#include "gossip_common.hpp"
#include "interact_run.hpp"
#include "lsq_wave.hpp"
#include "uniform_address.hpp"

namespace swarm {

constexpr int RUN_COLS = 128;                     // columns per workgroup
constexpr int TEAMS = 4;                          // waves per workgroup, each with interactions of its own
constexpr uint32_t RUN_LSQ_NODES = 64;            // 64 KiB of local memory
constexpr uint32_t RUN_LSQ_WORDS = 2048;          // batch x workgroups: every wave reads so many words per step
constexpr uint64_t WAIT_TICKS = 200000000ull;     // 2 s of the 100 MHz wall clock

struct LsqRunArgs {
    GossipArgs g;
    const RunDesc *descs;     // device, or null: the single interaction `one`
    RunDesc one;
    const float *A, *b;
    float *W;
    unsigned long long *part; // [team][step parity][workgroup][NB] words (tag << 32 | float bits)
    uint32_t count, m_rows, batch, tag;       // tag: of a team's first step
    float lr;
};

typedef float f2v __attribute__((ext_vector_type(2)));

// Two columns of a row of codes: BITS bits each.
template <int BITS>
__device__ __forceinline__ void store_code_pair(uint8_t *row, uint64_t col, uint32_t z0, uint32_t z1, bool in) {
    constexpr uint32_t MASK = (uint32_t)((1ull << BITS) - 1);
    const uint32_t c = (z0 & MASK) | ((z1 & MASK) << (BITS & 31));
    if constexpr (BITS == 2) {                    // half a byte: the even lane stores its neighbour's as well
        const uint32_t next = (uint32_t)__shfl_xor((int)c, 1);
        if (in && (threadIdx.x & 1u) == 0) row[col / 4] = (uint8_t)(c | (next << 4));
    } else if (in) {
        if constexpr (BITS == 4) row[col / 2] = (uint8_t)c;
        if constexpr (BITS == 8) *(uint16_t *)(row + col) = (uint16_t)c;
        if constexpr (BITS == 16) *(uint32_t *)(row + 2 * col) = c;
    }
}

// NB: the batch rounded up to 16 or 32 rows (64 would not leave the registers to request the next step's rows).
template <int BITS, int NB>
__global__ __launch_bounds__(TEAMS * 64, 1) void lsq_run_kernel(const LsqRunArgs ra) {
    extern __shared__ f2v models[];               // n x 64 pairs of columns of X, then the same of Xhat
    __shared__ uint32_t done[RUN_LSQ_NODES];      // interactions each node has been through
    __shared__ uint32_t bail;
    const GossipArgs &a = ra.g;
    const uint32_t lane = threadIdx.x & 63u, team = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t group = blockIdx.x, groups = gridDim.x, n = a.n, batch = ra.batch;
    const uint64_t d = a.d, col = (uint64_t)group * RUN_COLS + 2u * lane;
    const bool in = col < d;
    const uint32_t at_col = in ? (uint32_t)col : 0u;        // lanes past the row read its first columns, and no sum or store takes them
    const f2v zero = {0.f, 0.f};
    f2v *const X = models, *const Xhat = models + n * 64u;
    const float step = ra.lr * ((float)ra.m_rows / (float)batch);

    auto desc = [&](uint32_t k) { return ra.descs ? run_desc(ra.descs, k, ra.count) : ra.one; };
    // the rows step q of an interaction draws: index and right-hand side of row s in lane s, the lane's columns in `rows`
    auto fetch = [&](const RunDesc &rd, uint32_t q, f2v rows[NB], float &rhs) {
        const uint32_t node = rd.nodes & 0xFFFFu;
        const Words4 r = stream(a.seed, TAG_BATCH, q, node, rd.event, (lane % NB) >> 2);
        const uint32_t word = (lane & 3u) == 0 ? r.w0 : (lane & 3u) == 1 ? r.w1 : (lane & 3u) == 2 ? r.w2 : r.w3;
        const uint32_t row = scaled_index(word, ra.m_rows);
        rhs = ra.b[(uint64_t)node * ra.m_rows + row];
        const float *An = ra.A + (uint64_t)node * ra.m_rows * d;
        auto take = [&](int s) {
            const uint32_t drawn = (uint32_t)__builtin_amdgcn_readlane((int)row, s);
            rows[s] = *(SWARM_GLOBAL const f2v *)at_bytes(uniform(An + (uint64_t)drawn * d), 4u * at_col);
        };
        if (batch == NB) {
#pragma unroll
            for (int s = 0; s < NB; ++s) take(s);
        } else {
#pragma unroll
            for (int s = 0; s < NB; ++s)
                if ((uint32_t)s < batch) take(s);
        }
    };

    if (threadIdx.x < n) done[threadIdx.x] = 0;
    if (threadIdx.x == 0) bail = 0;
    f2v rows[NB] = {}, rows_next[NB] = {};
    float rhs = 0.f, rhs_next = 0.f;
    RunDesc next = desc(team);
    if (team < ra.count) fetch(next, 0, rows, rhs);
    const bool single = !ra.descs;                // a single interaction touches two nodes
    for (uint32_t u = team; u < (single ? 2u : n); u += TEAMS) {
        const uint32_t node = single ? (u ? ra.one.nodes >> 16 : ra.one.nodes & 0xFFFFu) : u;
        const f2v x = *(const f2v *)(a.X + (uint64_t)node * d + at_col), h = *(const f2v *)(a.Xhat + (uint64_t)node * d + at_col);
        X[node * 64u + lane] = in ? x : zero;
        Xhat[node * 64u + lane] = in ? h : zero;
    }
    __syncthreads();

    uint32_t turn_of_step = 0;                    // steps this team has taken: numbers the exchanged words
    bool clamped = false, lost = false;
    int fails = 0;
    for (uint32_t k = team; k < ra.count && !lost; k += TEAMS) {
        const RunDesc rd = next;
        next = desc(k + TEAMS);
        const uint32_t ni = rd.nodes & 0xFFFFu, nj = rd.nodes >> 16, H = (rd.flags >> 8) & 0xFFu;
        const uint64_t t0 = wall_clock64();
        while ((first_lane(__hip_atomic_load(&done[ni], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) ^ (rd.turn & 0xFFFFu)) |
               (first_lane(__hip_atomic_load(&done[nj], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) ^ (rd.turn >> 16))) {
            lost = first_lane(__hip_atomic_load(&bail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0 ||
                   wall_clock64() - t0 > WAIT_TICKS;
            if (lost) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (lost) break;
        const f2v h = Xhat[ni * 64u + lane];
        f2v w = h;
        for (uint32_t q = 0; q < H && !lost; ++q) {
            float dots[NB];
#pragma unroll
            for (int s = 0; s < NB; ++s) dots[s] = in ? fmaf(rows[s].y, w.y, rows[s].x * w.x) : 0.f;
            const float share = wave_totals<NB>(dots, lane);
            const uint32_t tag = ra.tag + turn_of_step;
            unsigned long long *words = ra.part + (uint64_t)(team * 2u + (turn_of_step & 1u)) * groups * NB;
            if (lane < NB)
                __hip_atomic_store(words + (uint64_t)group * NB + lane, ((unsigned long long)tag << 32) | __float_as_uint(share),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool more = q + 1 < H;
            if (more || k + TEAMS < ra.count) fetch(more ? rd : next, more ? q + 1 : 0u, rows_next, rhs_next);
            // the residual of row lane % NB: lanes with the same row take every (64 / NB)-th workgroup's share, in order
            float residual = 0.f;
            const uint64_t t1 = wall_clock64();
            auto collect = [&](auto requests) {           // `requests` words per lane at a time
                constexpr uint32_t WORDS = decltype(requests)::value;
                for (uint32_t g0 = 0; g0 < groups && !lost; g0 += WORDS * (64u / NB)) {
                    unsigned long long word[WORDS];
                    while (true) {
                        bool here = true;
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i) {
                            const uint32_t from = g0 + (64u / NB) * i + lane / NB;
                            word[i] = __hip_atomic_load(words + (uint64_t)min(from, groups - 1u) * NB + lane % NB, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
                        }
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i) here &= (uint32_t)(word[i] >> 32) == tag;
                        if (__all(here)) break;
                        lost = first_lane(__hip_atomic_load(&bail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0 ||
                               wall_clock64() - t1 > WAIT_TICKS;
                        if (lost) break;
                    }
#pragma unroll
                    for (uint32_t i = 0; i < WORDS; ++i)
                        residual += g0 + (64u / NB) * i + lane / NB < groups ? __uint_as_float((uint32_t)word[i]) : 0.f;
                }
            };
            if (groups <= 8u * (64u / NB)) collect(std::integral_constant<uint32_t, 8>{});
            else collect(std::integral_constant<uint32_t, 16>{});
#pragma unroll
            for (int off = NB; off < 64; off *= 2) residual += __shfl_xor(residual, off);
            residual -= rhs;
            f2v parts[4] = {zero, zero, zero, zero};      // of every fourth row: a chain of NB rounds more (2.78e-8 off 64 bits after 200 interactions, 2.68e-8 so) and takes 1 % longer
#pragma unroll
            for (int s = 0; s < NB; ++s) {
                const float r = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residual), s));
                f2v &p = parts[s & 3];
                if ((uint32_t)s < batch) { p.x = fmaf(rows[s].x, r, p.x); p.y = fmaf(rows[s].y, r, p.y); }
            }
            const f2v g = (parts[0] + parts[1]) + (parts[2] + parts[3]);
            w.x = fmaf(-step, g.x, w.x);
            w.y = fmaf(-step, g.y, w.y);
#pragma unroll
            for (int s = 0; s < NB; ++s) rows[s] = rows_next[s];
            rhs = rhs_next;
            ++turn_of_step;
        }
        if (lost) break;
        const f2v xi = X[ni * 64u + lane], xj = X[nj * 64u + lane];
        f2v average;
        if constexpr (BITS > 0) {
            // a call of the generator serves 8 columns: word (column / 2) % 4, low half first
            const Words4 wi = stream(a.seed, TAG_SR, 0, ni, rd.event, col / 8), wj = stream(a.seed, TAG_SR, 0, nj, rd.event, col / 8);
            const uint32_t ri = (lane & 3u) == 0 ? wi.w0 : (lane & 3u) == 1 ? wi.w1 : (lane & 3u) == 2 ? wi.w2 : wi.w3;
            const uint32_t rj = (lane & 3u) == 0 ? wj.w0 : (lane & 3u) == 1 ? wj.w1 : (lane & 3u) == 2 ? wj.w2 : wj.w3;
            constexpr uint32_t MASK = (uint32_t)((1ull << BITS) - 1);
            const float half_eps = 0.5f * a.eps;
            bool far = false;
            const int zi0 = stochastic_round(xi.x, a.inv_eps, ri & 0xFFFFu, far), zi1 = stochastic_round(xi.y, a.inv_eps, ri >> 16, far);
            const int zj0 = stochastic_round(xj.x, a.inv_eps, rj & 0xFFFFu, far), zj1 = stochastic_round(xj.y, a.inv_eps, rj >> 16, far);
            const int p0 = decode_near<BITS>((uint32_t)zj0 & MASK, key_cell(xi.x, a.inv_eps, far));
            const int p1 = decode_near<BITS>((uint32_t)zj1 & MASK, key_cell(xi.y, a.inv_eps, far));
            fails += in ? (p0 != zj0) + (p1 != zj1) : 0;
            clamped |= in && far;
            average.x = fmaf((float)(zi0 + p0), half_eps, 0.f);
            average.y = fmaf((float)(zi1 + p1), half_eps, 0.f);
            if (rd.flags & RUN_LAST_OF_I) store_code_pair<BITS>(a.ring + (uint64_t)ni * a.row_bytes, col, (uint32_t)zi0, (uint32_t)zi1, in);
            if (rd.flags & RUN_LAST_OF_J) store_code_pair<BITS>(a.ring + (uint64_t)nj * a.row_bytes, col, (uint32_t)zj0, (uint32_t)zj1, in);
        } else {
            average = 0.5f * (xi + xj);
        }
        const f2v out = average + (w - h);
        X[ni * 64u + lane] = out;
        Xhat[ni * 64u + lane] = out;
        X[nj * 64u + lane] = average;
        if ((rd.flags & RUN_LAST_LED) && in) *(f2v *)(ra.W + (uint64_t)ni * d + col) = w;
        __hip_atomic_store(&done[ni], (rd.turn & 0xFFFFu) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&done[nj], (rd.turn >> 16) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (lost) {
        __hip_atomic_store(&bail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (lane == 0) atomicOr(&a.counters->barrier_timeouts, 1u);
    }
    if (BITS > 0) report(a.counters, fails, clamped);
    __syncthreads();
    if (bail) return;                             // as far as it got is no state to keep
    for (uint32_t u = team; u < n; u += TEAMS)
        if (done[u] != 0 && in) {
            *(f2v *)(a.X + (uint64_t)u * d + col) = X[u * 64u + lane];
            *(f2v *)(a.Xhat + (uint64_t)u * d + col) = Xhat[u * 64u + lane];
        }
}

bool lsq_run_fits(uint64_t d, uint32_t n, uint32_t batch) {
    return n <= RUN_LSQ_NODES && (d + RUN_COLS - 1) / RUN_COLS * batch <= RUN_LSQ_WORDS && (d + RUN_COLS - 1) / RUN_COLS <= 64 && batch <= 32;
}

static uint32_t padded_batch(uint32_t batch) { return batch <= 16 ? 16 : 32; }

size_t lsq_run_bytes(uint64_t d, uint32_t batch) {
    return sizeof(unsigned long long) * TEAMS * 2 * ((d + RUN_COLS - 1) / RUN_COLS) * padded_batch(batch);
}

template <int BITS>
static void launch_batch(const LsqRunArgs &ra, uint32_t groups, hipStream_t st) {
    const size_t lds = (size_t)ra.g.n * 128 * sizeof(f2v);
    if (ra.batch <= 16) lsq_run_kernel<BITS, 16><<<groups, TEAMS * 64, lds, st>>>(ra);
    else lsq_run_kernel<BITS, 32><<<groups, TEAMS * 64, lds, st>>>(ra);
}

// total_steps: of all interactions of the launch together.
hipError_t launch_lsq_run(const GossipArgs &g, uint32_t bits, const RunDesc *descs_dev, RunDesc one, uint32_t count,
                          uint32_t total_steps, LsqObjective &o, float lr, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!o.run_part) return hipErrorInvalidValue;
    if (o.run_tag > 0xFFFFFFFEu - total_steps) {         // tags would wrap: start over on wiped words, in stream order
        const hipError_t e = hipMemsetAsync(o.run_part, 0xFF, o.run_part_bytes, st);
        if (e != hipSuccess) return e;
        o.run_tag = 0;
    }
    const LsqRunArgs ra{g, descs_dev, one, o.A, o.b, const_cast<float *>(g.W), o.run_part, count, o.m_rows, o.batch, o.run_tag, lr};
    o.run_tag += total_steps;
    const uint32_t groups = (uint32_t)((g.d + RUN_COLS - 1) / RUN_COLS);
    switch (bits) {
        case 0: launch_batch<0>(ra, groups, st); break;
        case 2: launch_batch<2>(ra, groups, st); break;
        case 4: launch_batch<4>(ra, groups, st); break;
        case 8: launch_batch<8>(ra, groups, st); break;
        case 16: launch_batch<16>(ra, groups, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace swarm
