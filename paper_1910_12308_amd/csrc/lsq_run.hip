// Algorithm 1 on small least-squares swarms: a run of interactions (or a single one) in one launch.  A workgroup owns
// 128 columns of all n models and snapshots and keeps them in local memory (1 KiB per node); each of its four teams of four
// waves takes every fourth interaction, in an order in which every interaction follows those it depends on, and waits in
// local memory for the earlier interactions of its two nodes (as in interact_run.hip).  A wave holds every fourth of the
// batch's rows of A, a lane two columns of them: the products need no other lane but for the residuals, and of those only
// the sums over a workgroup's columns leave it.  The waves that hold the same rows in the other workgroups wait for these
// words in device memory, each tagged with the number of its step, so that nothing has to be cleared between steps; two
// sets of words alternate, because a wave writes its words of step c + 2 after it has read all words of step c + 1, and
// those were written by waves that had read step c.  The gradients of a team's waves meet in local memory (two sets of
// them for the same reason), and every wave applies their sum to a copy of the model of its own.
// Bound by latency: interactions that share a node follow one another, and a step is a chain of products, sums over the
// wave, one exchange through device memory, one through local memory and an update.  So whatever needs no model is done
// before the wait for the nodes (the random words, by one call of the generator per lane, and the rows of two steps) or
// while the words travel (the pair's average), and the rows are split between waves (one wave took 4200 of a step's 9600
// cycles to draw and request 32 rows).  What is left, in cycles at 8 nodes x 4096, batch 32: 600 products and sums, 3500 until
// the words are there, 400 gradient, 900 until the team's have met.  Words that are asked for too early hold up the stores they wait
// for: hence the pause, and requests for what is missing only.  200 interactions, H = 2: 593 us, 979 with one wave per team;
// 8 x 1024, batch 16: 400 and 649; a single interaction 10.7 us and 13.6 (8 x 8192).  With a pause of 256
// cycles 657, and 426 instead of 380 at 2048 columns, batch 16.  All workgroups on one die: no faster (4 % at 8 workgroups, slower at 32).
// Four teams per workgroup are room for four interactions side by side: graphs that let many more run at once keep a launch
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
constexpr int TEAMS = 4;                          // per workgroup, each with interactions of its own
constexpr int CREW = 4;                           // waves of a team, each with rows of its own
constexpr uint32_t RUN_LSQ_NODES = 64;            // 64 KiB of local memory
constexpr uint32_t RUN_LSQ_WORDS = 2048;          // batch x workgroups: a team reads so many words per step, each wave a quarter
constexpr uint64_t WAIT_TICKS = 200000000ull;     // 2 s of the 100 MHz wall clock

struct LsqRunArgs {
    GossipArgs g;
    const RunDesc *descs;     // device, or null: the single interaction `one`
    RunDesc one;
    const float *A, *b;
    float *W;
    unsigned long long *part; // [team][step parity][wave][workgroup][row] words (tag << 32 | float bits)
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

// Workgroups a row has words for: whole requests of a wave (R rows of CREW * 64 / NB workgroups), a power of two of them.
__host__ __device__ __forceinline__ uint32_t slots_of(uint32_t groups, uint32_t padded) {
    uint32_t slots = CREW * 64 / padded;
    while (slots < groups) slots *= 2;
    return slots;
}

// A word at a lane's and a uniform offset, as other workgroups' stores left it (SC1: past this die's caches).
__device__ __forceinline__ unsigned long long word_of_agent(__amdgpu_buffer_rsrc_t words, uint32_t lane_offset, uint32_t offset) {
    constexpr int SC1 = 16;
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(words, (int)lane_offset, (int)offset, SC1);
    return (unsigned long long)v[1] << 32 | v[0];
}

// NB: the batch rounded up to 16 or 32 rows.
template <int BITS, int NB>
__global__ __launch_bounds__(TEAMS * CREW * 64, 1) void lsq_run_kernel(const LsqRunArgs ra) {
    constexpr int R = NB / CREW;                  // rows of a wave
    constexpr int WAVES = TEAMS * CREW;
    constexpr uint32_t STEPS = 32 / R;            // whose rows a call of the generator per lane draws
    extern __shared__ f2v models[];               // n x 64 pairs of columns of X, then the same of Xhat
    __shared__ uint32_t done[RUN_LSQ_NODES];      // interactions each node has been through
    __shared__ f2v shares[TEAMS][2][CREW][64];    // of the gradient, by step parity
    __shared__ __attribute__((aligned(16))) uint32_t arrived[TEAMS][CREW];     // steps whose share a wave has left
    __shared__ uint32_t bail;
    const GossipArgs &a = ra.g;
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t team = wave / CREW, mate = wave % CREW, at_row = lane / CREW % R;
    const uint32_t group = blockIdx.x, groups = gridDim.x, n = a.n, own = ra.batch / CREW;        // the batch is a multiple of 4
    const uint64_t d = a.d, col = (uint64_t)group * RUN_COLS + 2u * lane;
    const bool in = col < d;
    const uint32_t at_col = in ? (uint32_t)col : 0u;        // lanes past the row read its first columns, and no sum or store takes them
    const f2v zero = {0.f, 0.f};
    f2v *const X = models, *const Xhat = models + n * 64u;
    constexpr uint32_t EACH = CREW * 64 / NB;     // workgroups whose words a request takes
    const uint32_t slots = slots_of(groups, NB), first = 64u / NB * (lane % CREW) + lane / NB, mine_from = 8u * (first * R + at_row);
    const auto part = __builtin_amdgcn_make_buffer_rsrc((void *)ra.part, 0, (int)(TEAMS * 2 * NB * 8u * slots), 0x00020000);
    // Cycles from a wave's words to its first request.  us for 200 interactions of 8 nodes, H = 2, at 256 / 768 / 1280 / 1792 cycles:
    // batch 32, 4096 columns 657 / 599 / 595 / 622, 1024: 466 / 431 / 463 / 508, 8192: 868 / 794 / 784 / 808, 128 (alone): 362 / 386 / 444 / 495;
    // batch 16, 2048: 426 / 380 / 429 / 479; 16 nodes x 8192, H = 1: 313 / 274 / 258 / 239.  By workgroups alone: with 64 of them
    // (1920 cycles) two steps at batch 32 pay for the single steps (8 nodes x 8192, H = 2: 780, 760 at 1280; 16 nodes, H = 1: 316 and
    // 324 at batch 32, 230 and 248 at batch 16).
    const uint64_t pause = groups == 1 ? 0u : 640u + 20u * groups;
    const float step = ra.lr * ((float)ra.m_rows / (float)ra.batch);

    uint64_t seed = a.seed;
    auto here = [](uint64_t v) {                  // what follows from v is worked out where it is used: its registers are short
        asm volatile("" : "+s"(v));
        return v;
    };

    auto desc = [&](uint32_t k) { return ra.descs ? run_desc(ra.descs, k, ra.count) : ra.one; };
    auto given_up = [&](uint64_t since) {
        return first_lane(__hip_atomic_load(&bail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0 || wall_clock64() - since > WAIT_TICKS;
    };

    if (threadIdx.x < n) done[threadIdx.x] = 0;
    if (threadIdx.x < WAVES) arrived[threadIdx.x / CREW][threadIdx.x % CREW] = 0;
    if (threadIdx.x == 0) bail = 0;
    f2v rows_even[R] = {}, rows_odd[R] = {};      // of even and odd steps
    float rhs_even = 0.f, rhs_odd = 0.f;
    uint32_t drawn = 0, ri = 0, rj = 0;           // rows of A, and random words of the pair's rounding
    // A wave's rows are every fourth of the batch's: row mate + 4 i.  One call of the generator per lane serves lanes 0..15 and
    // 16..31 with the random words of the pair's rounding, the other lanes with the rows of A that STEPS steps from the first draw.
    auto draw = [&](const RunDesc &rd, uint32_t q) {
        const uint32_t ni = rd.nodes & 0xFFFFu, nj = rd.nodes >> 16;
        const bool rows = lane >= 32;
        const Words4 r = stream(here(seed), rows ? TAG_BATCH : TAG_SR, rows ? q + (lane - 32u) / R : 0u, rows || lane < 16 ? ni : nj, rd.event,
                                rows ? lane % R : 16u * group + lane % 16u);
        drawn = scaled_index(mate == 0 ? r.w0 : mate == 1 ? r.w1 : mate == 2 ? r.w2 : r.w3, ra.m_rows);
        return r;
    };
    // the lane's columns of step q's rows (past the batch of rows that no sum takes), and the right-hand side of row `at_row`
    auto request = [&](const RunDesc &rd, uint32_t q, f2v (&rows)[R], float &rhs) {
        const uint32_t node = rd.nodes & 0xFFFFu, from = 32u + R * (q % STEPS);
        const uint32_t row = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (from + at_row)), (int)drawn);
        const uint64_t row_at = (uint64_t)(ra.A + (uint64_t)node * ra.m_rows * d) + (uint64_t)drawn * (4u * d);
        uint32_t offset = 4u * at_col;
        asm("" : "+v"(offset));                   // a 32-bit offset to a scalar base, not a 64-bit one made ahead of the loop
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t low = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)row_at, from + i);
            const uint32_t high = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(row_at >> 32), from + i);
            rows[i] = *(SWARM_GLOBAL const f2v *)at_bytes(uniform((const float *)((uint64_t)high << 32 | low)), offset);
        }
        rhs = ra.b[(uint64_t)node * ra.m_rows + row];
    };
    auto prepare = [&](const RunDesc &rd) {
        const Words4 r = draw(rd, 0);
        request(rd, 0, rows_even, rhs_even);
        if (((rd.flags >> 8) & 0xFFu) > 1) request(rd, 1, rows_odd, rhs_odd);
        if (BITS > 0 && mate == 0) {              // a call serves 8 columns: word (column / 2) % 4, low half first
            auto word_of = [&](uint32_t call) {
                const uint32_t w0 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * call), (int)r.w0);
                const uint32_t w1 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * call), (int)r.w1);
                const uint32_t w2 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * call), (int)r.w2);
                const uint32_t w3 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * call), (int)r.w3);
                return (lane & 3u) == 0 ? w0 : (lane & 3u) == 1 ? w1 : (lane & 3u) == 2 ? w2 : w3;
            };
            ri = word_of(lane / 4u);
            rj = word_of(16u + lane / 4u);
        }
    };
    RunDesc next = desc(team);
    if (team < ra.count) prepare(next);
    const bool single = !ra.descs;                // a single interaction touches two nodes
    for (uint32_t u = wave; u < (single ? 2u : n); u += WAVES) {
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
        while (true) {                            // both nodes' earlier interactions
            const uint32_t turn = __hip_atomic_load(&done[lane & 1u ? nj : ni], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (__all(turn == (lane & 1u ? rd.turn >> 16 : rd.turn & 0xFFFFu))) break;
            lost = given_up(t0);
            if (lost) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (lost) break;
        __builtin_amdgcn_s_setprio(2);            // ahead of the teams that wait
        const f2v h = Xhat[ni * 64u + lane], xi = X[ni * 64u + lane], xj = X[nj * 64u + lane];
        f2v w = h, average = zero;
        int zi0 = 0, zi1 = 0, zj0 = 0, zj1 = 0;
        auto meet = [&] {                         // the pair's average takes no local step
            if constexpr (BITS > 0) {
                constexpr uint32_t MASK = (uint32_t)((1ull << BITS) - 1);
                const float half_eps = 0.5f * a.eps;
                bool far = false;
                zi0 = stochastic_round(xi.x, a.inv_eps, ri & 0xFFFFu, far), zi1 = stochastic_round(xi.y, a.inv_eps, ri >> 16, far);
                zj0 = stochastic_round(xj.x, a.inv_eps, rj & 0xFFFFu, far), zj1 = stochastic_round(xj.y, a.inv_eps, rj >> 16, far);
                const int p0 = decode_near<BITS>((uint32_t)zj0 & MASK, key_cell(xi.x, a.inv_eps, far));
                const int p1 = decode_near<BITS>((uint32_t)zj1 & MASK, key_cell(xi.y, a.inv_eps, far));
                fails += in ? (p0 != zj0) + (p1 != zj1) : 0;
                clamped |= in && far;
                average.x = fmaf((float)(zi0 + p0), half_eps, 0.f);
                average.y = fmaf((float)(zi1 + p1), half_eps, 0.f);
            } else {
                average = 0.5f * (xi + xj);
            }
        };
        auto take_step = [&](uint32_t q, f2v (&rows)[R], float &rhs) {
            float dots[R];
#pragma unroll
            for (int i = 0; i < R; ++i) dots[i] = in ? fmaf(rows[i].y, w.y, rows[i].x * w.x) : 0.f;
            const float share = wave_totals<R, NB / 2>(dots, lane);
            const uint32_t tag = ra.tag + turn_of_step;
            const uint32_t set = ((team * 2u + (turn_of_step & 1u)) * CREW + mate) * slots * (R * 8u);
            if (lane < NB && lane % CREW == 0)
                __hip_atomic_store(ra.part + (set / 8u + group * R + at_row), ((unsigned long long)tag << 32) | __float_as_uint(share),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t published = __builtin_readcyclecounter();
            // while the words travel
            if (q == 0 && mate == 0) meet();
            const bool again = q + 2 < H;
            if (again && (q + 2) % STEPS == 0) draw(rd, q + 2);
            // the residual of row `at_row`: the shares of the workgroups lane / NB, lane / NB + 64 / NB .., in order, requested by
            // the quad's lanes in turn, then the sum of these sums
            float residual = 0.f;
            while (__builtin_readcyclecounter() - published < pause) __builtin_amdgcn_s_sleep(1);
            const uint64_t t1 = wall_clock64();
            auto collect = [&](auto requests) {           // `requests` words per lane at a time
                constexpr uint32_t WORDS = decltype(requests)::value;
                for (uint32_t g0 = 0; g0 < groups && !lost; g0 += WORDS * EACH) {
                    unsigned long long word[WORDS];
                    auto ask = [&](uint32_t i) { word[i] = word_of_agent(part, mine_from, set + (g0 + i * EACH) * (R * 8u)); };
                    auto missing = [&](uint32_t i) {
                        return !__all((uint32_t)(word[i] >> 32) == tag || g0 + i * EACH + first >= groups);
                    };
                    asm volatile("" ::: "memory");        // not before the pause
#pragma unroll
                    for (uint32_t i = 0; i < WORDS; ++i) ask(i);
                    while (true) {
                        uint32_t late = 0;
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i) late |= missing(i) ? 1u << i : 0u;
                        if (late == 0) break;
                        lost = given_up(t1);
                        if (lost) break;
                        __builtin_amdgcn_s_sleep(1);
                        asm volatile("" ::: "memory");    // what is read again
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i)
                            if (late & 1u << i) ask(i);
                    }
#pragma unroll
                    for (uint32_t i = 0; i < WORDS; ++i) {
                        const int v = g0 + i * EACH + first < groups ? (int)(uint32_t)word[i] : 0;
                        residual += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(v, 0x00, 0xF, 0xF, true));   // of the quad's lane 0
                        residual += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(v, 0x55, 0xF, 0xF, true));
                        residual += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(v, 0xAA, 0xF, 0xF, true));
                        residual += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(v, 0xFF, 0xF, 0xF, true));
                    }
                }
            };
            if (slots == EACH) collect(std::integral_constant<uint32_t, 1>{});
            else if (slots == 2 * EACH) collect(std::integral_constant<uint32_t, 2>{});
            else collect(std::integral_constant<uint32_t, 4>{});
            residual = total_from<NB>(residual, lane);
            residual -= rhs;
            f2v share_of_g = zero;                        // of every fourth row: one chain of all rounds more (2.78e-8 off 64 bits after 200 interactions, 2.68e-8 so)
            auto add = [&](int i) {
                const float r = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residual), CREW * i));
                share_of_g.x = fmaf(rows[i].x, r, share_of_g.x);
                share_of_g.y = fmaf(rows[i].y, r, share_of_g.y);
            };
            if (own == R) {
#pragma unroll
                for (int i = 0; i < R; ++i) add(i);
            } else {
#pragma unroll
                for (int i = 0; i < R; ++i)
                    if ((uint32_t)i < own) add(i);
            }
            // the team's shares meet: a wave's words reach local memory in order, and the next set is not written before every mate
            // has read this one
            f2v (*mine)[64] = shares[team][turn_of_step & 1u];
            mine[mate][lane] = share_of_g;
            __hip_atomic_store(&arrived[team][mate], ++turn_of_step, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (again) request(rd, q + 2, rows, rhs);
            while (true) {
                const uint32_t steps = __hip_atomic_load(&arrived[team][lane % CREW], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (__all(steps - turn_of_step <= 1u)) break;
                lost = lost || given_up(t1);
                if (lost) break;
            }
            const f2v g = (mine[0][lane] + mine[1][lane]) + (mine[2][lane] + mine[3][lane]);
            w.x = fmaf(-step, g.x, w.x);
            w.y = fmaf(-step, g.y, w.y);
        };
        for (uint32_t q = 0; q < H && !lost; q += 2) {
            take_step(q, rows_even, rhs_even);
            if (q + 1 < H && !lost) take_step(q + 1, rows_odd, rhs_odd);
        }
        if (lost) break;
        if (mate == 0) {                          // a team's first wave finishes the interaction; the others meet it at `done`
            const f2v out = average + (w - h);
            X[ni * 64u + lane] = out;
            Xhat[ni * 64u + lane] = out;
            X[nj * 64u + lane] = average;
            __hip_atomic_store(&done[ni], (rd.turn & 0xFFFFu) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(&done[nj], (rd.turn >> 16) + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if constexpr (BITS > 0) {
                if (rd.flags & RUN_LAST_OF_I) store_code_pair<BITS>(a.ring + (uint64_t)ni * a.row_bytes, col, (uint32_t)zi0, (uint32_t)zi1, in);
                if (rd.flags & RUN_LAST_OF_J) store_code_pair<BITS>(a.ring + (uint64_t)nj * a.row_bytes, col, (uint32_t)zj0, (uint32_t)zj1, in);
            }
            if ((rd.flags & RUN_LAST_LED) && in) *(f2v *)(ra.W + (uint64_t)ni * d + col) = w;
        }
        __builtin_amdgcn_s_setprio(0);
        if (k + TEAMS < ra.count) prepare(next);
    }
    if (lost) {
        __hip_atomic_store(&bail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (lane == 0) atomicOr(&a.counters->barrier_timeouts, 1u);
    }
    if (BITS > 0) report(a.counters, fails, clamped);
    __syncthreads();
    if (bail) return;                             // as far as it got is no state to keep
    for (uint32_t u = wave; u < n; u += WAVES)
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
    return sizeof(unsigned long long) * TEAMS * 2 * slots_of((uint32_t)((d + RUN_COLS - 1) / RUN_COLS), padded_batch(batch)) * padded_batch(batch);
}

template <int BITS>
static void launch_batch(const LsqRunArgs &ra, uint32_t groups, hipStream_t st) {
    const size_t lds = (size_t)ra.g.n * 128 * sizeof(f2v);
    if (ra.batch <= 16) lsq_run_kernel<BITS, 16><<<groups, TEAMS * CREW * 64, lds, st>>>(ra);
    else lsq_run_kernel<BITS, 32><<<groups, TEAMS * CREW * 64, lds, st>>>(ra);
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
