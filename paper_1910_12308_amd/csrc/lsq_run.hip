// Algorithm 1 on small least-squares swarms: a run of interactions (or a single one) in one launch.  A workgroup owns
// 128 columns of all n models and snapshots and keeps them in local memory (1 KiB per node).  The local steps of an interaction
// need the initiator's snapshot and nothing else of the interactions before it, so they are taken apart from it: seven teams
// of two waves take the steps of every seventh interaction as soon as the initiator's last interaction of its own has ended,
// and one wave takes the interactions in their order, each when its steps are there.  So the chain of interactions that share
// a node is a chain of averages, and only the interactions that a node leads wait for one another's steps.
// A wave holds every second of the batch's rows of A, a lane two columns of them: the products need no other lane but for the
// residuals, and of those only the sums over a workgroup's columns leave it.  The waves that hold the same rows in the other
// workgroups wait for these words in device memory, each tagged with the number of its step, so that nothing has to be cleared
// between steps; two sets of words alternate, because a wave writes its words of step c + 2 after it has read all words of step
// c + 1, and those were written by waves that had read step c.  The gradients of a team's waves meet in local memory (two sets of
// them for the same reason), and every wave applies their sum to a copy of the model of its own.
// Bound by latency: a step is a chain of products, sums over the wave, one exchange through device memory, one through local
// memory and an update.  So what needs no model is done before the wait for the snapshot (an interaction's rows are drawn by one
// call of the generator per lane, and those of its first two steps requested) or while the words travel (the rows of later steps).
// In cycles per step at 8 nodes x 4096, batch 32: 500 products and sums, 3800 until the words of all 32 workgroups are there (2300
// with 8), 500 gradient, 700 until the team's two have met.  Words that are asked for too early hold up the stores they wait for:
// hence the pause, and requests for what is missing only.
// us for 200 interactions on a complete graph, against teams of four waves that each kept an interaction from its wait for both
// nodes to its end (four side by side):
//   8 x 4096, batch 32, H = 2    593  364      8 x 1024, batch 32, H = 2    444  291     12 x 2048, batch 16, H = 3    458  296
//   8 x 8192, batch 32, H = 1    439  269     16 x 8192, batch 32, H = 2    603  339
// A single interaction of 8 x 8192, batch 32, H = 2: 10.6 and 10.3.  Five teams instead of seven: 375, and 392 at 16 x 8192.  An
// interaction's rows requested during the last steps of the one before: 383 and 378.
// All workgroups are resident together (at most 64), the earliest unfinished interaction waits for none, and every
// wait is bounded, so that all waves end whatever happens to the others.
#include <type_traits>

#include "gossip_common.hpp"
#include "interact_run.hpp"
#include "lsq_wave.hpp"
#include "uniform_address.hpp"

namespace swarm {

constexpr int RUN_COLS = 128;                     // columns per workgroup
constexpr int CREW = 2;                           // waves of a team, each with rows of its own
constexpr int TEAMS = 7;                          // per workgroup, each with steps of its own
constexpr int RUN_WAVES = TEAMS * CREW + 1;       // the last one takes the interactions
constexpr uint32_t RUN_LSQ_NODES = 64;            // 64 KiB of local memory
constexpr uint32_t RUN_LSQ_WORDS = 2048;          // batch x workgroups: a team reads so many words per step, each wave half of them
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

// Workgroups that a set has words for: whole requests of a wave (64 words).
__host__ __device__ __forceinline__ uint32_t slots_of(uint32_t groups, uint32_t padded) {
    const uint32_t each = CREW * 64 / padded;
    return (groups + each - 1) / each * each;
}

// A word at a lane's and a uniform offset, as other workgroups' stores left it (SC1: past this die's caches).
__device__ __forceinline__ unsigned long long word_of_agent(__amdgpu_buffer_rsrc_t words, uint32_t lane_offset, uint32_t offset) {
    constexpr int SC1 = 16;
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(words, (int)lane_offset, (int)offset, SC1);
    return (unsigned long long)v[1] << 32 | v[0];
}

// NB: the batch rounded up to 16 or 32 rows.
template <int BITS, int NB>
__global__ __launch_bounds__(RUN_WAVES * 64, 1) void lsq_run_kernel(const LsqRunArgs ra) {
    constexpr int R = NB / CREW;                  // rows of a wave
    constexpr uint32_t EACH = 64 / R;             // steps whose rows a call of the generator per lane draws; workgroups whose words a request takes
    extern __shared__ f2v models[];               // n x 64 pairs of columns of X, then the same of Xhat
    __shared__ f2v shares[TEAMS][2][CREW][64];    // of the gradient, by step parity
    __shared__ f2v deltas[TEAMS][64];             // what the steps of a team's interaction have come to
    __shared__ uint32_t arrived[TEAMS][CREW];     // steps whose share a wave has left
    __shared__ uint32_t stepped[TEAMS];           // interactions whose steps a team has taken
    __shared__ uint32_t touched[RUN_LSQ_NODES];
    __shared__ uint32_t finished, bail;           // finished: interactions that have ended
    const GossipArgs &a = ra.g;
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t group = blockIdx.x, groups = gridDim.x, n = a.n;
    const uint64_t d = a.d, col = (uint64_t)group * RUN_COLS + 2u * lane;
    const bool in = col < d;
    const uint32_t at_col = in ? (uint32_t)col : 0u;        // lanes past the row read its first columns, and no sum or store takes them
    const f2v zero = {0.f, 0.f};
    f2v *const X = models, *const Xhat = models + n * 64u;

    uint64_t seed = a.seed;
    auto here = [](uint64_t v) {                  // what follows from v is worked out where it is used: its registers are short
        asm volatile("" : "+s"(v));
        return v;
    };
    auto desc = [&](uint32_t k) { return ra.descs ? run_desc(ra.descs, k, ra.count) : ra.one; };
    auto read = [](uint32_t *word) { return first_lane(__hip_atomic_load(word, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)); };
    auto post = [](uint32_t *word, uint32_t v) { __hip_atomic_store(word, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto given_up = [&](uint64_t since) {
        return first_lane(__hip_atomic_load(&bail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0 || wall_clock64() - since > WAIT_TICKS;
    };
    bool lost = false, clamped = false;
    int fails = 0;
    auto wait_for = [&](uint32_t *word, uint32_t least) {     // counts, far from wrapping
        if (read(word) >= least) return;
        const uint64_t t0 = wall_clock64();
        do {
            lost = lost || given_up(t0);
            if (lost) return;
            __builtin_amdgcn_s_sleep(1);
        } while (read(word) < least);
    };

    if (ra.descs && threadIdx.x < ra.count)       // on the way to this die's cache: whoever reads them there waits for little else
        asm volatile("" ::"v"(ra.descs[threadIdx.x].turn));
    if (threadIdx.x < n) touched[threadIdx.x] = 0;
    if (threadIdx.x < TEAMS) arrived[threadIdx.x][0] = arrived[threadIdx.x][1] = stepped[threadIdx.x] = 0;
    if (threadIdx.x == 0) finished = bail = 0;
    const bool single = !ra.descs;                // a single interaction touches two nodes
    const uint32_t team = wave / CREW, mate = wave % CREW;
    uint64_t row_at = 0;                          // rows of A and their right-hand sides, as drawn
    float rhs_at = 0.f;
    // A wave's rows are every second of the batch's: row mate + 2 i, of the steps q + lane / R
    auto draw = [&](const RunDesc &rd, uint32_t q) {
        const uint32_t i = lane % R, word = mate + 2u * (i & 1u), node = rd.nodes & 0xFFFFu;
        const Words4 r = stream(here(seed), TAG_BATCH, q + lane / R, node, rd.event, i >> 1);
        const uint64_t row = (uint64_t)node * ra.m_rows + scaled_index(word == 0 ? r.w0 : word == 1 ? r.w1 : word == 2 ? r.w2 : r.w3, ra.m_rows);
        row_at = (uint64_t)ra.A + 4u * row * d;
        rhs_at = ra.b[row];
    };
    // the lane's columns of the step's rows (past the batch of rows that no sum takes)
    auto request = [&](uint32_t q, f2v (&rows)[R]) {
        const uint32_t from = R * (q % EACH);
        uint32_t offset = 4u * at_col;
        asm("" : "+v"(offset));                   // a 32-bit offset to a scalar base, not a 64-bit one made ahead of the loop
        constexpr int B = 4;                      // addresses side by side: a scalar that a lane was read into may address a load five instructions later
#pragma unroll
        for (int i = 0; i < R; i += B) {
            uint64_t at[B];
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const uint32_t low = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)row_at, from + i + j);
                const uint32_t high = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(row_at >> 32), from + i + j);
                at[j] = (uint64_t)high << 32 | low;
            }
            asm volatile("" : "+s"(at[0]), "+s"(at[1]), "+s"(at[2]), "+s"(at[3]));
#pragma unroll
            for (int j = 0; j < B; ++j) rows[i + j] = *(SWARM_GLOBAL const f2v *)at_bytes((SWARM_GLOBAL const float *)at[j], offset);
        }
    };
    f2v rows[R] = {}, rows_ahead[R] = {};         // of this step and the next
    // Its rows come with the models, which other waves fetch, not after them (us of a call among others: 8 nodes x 1024, batch 16,
    // H = 1 5.8 -> 5.4, 32 x 512, batch 16, H = 2 7.1 -> 6.4); of a run the first wait for its descriptors.
    if (single && team == 0) {
        draw(ra.one, 0);
        request(0, rows);
        if (((ra.one.flags >> 8) & 0xFFu) > 1) request(1, rows_ahead);
    }
    for (uint32_t u = (wave + RUN_WAVES - CREW) % RUN_WAVES; u < (single ? 2u : n); u += RUN_WAVES) {
        const uint32_t node = single ? (u ? ra.one.nodes >> 16 : ra.one.nodes & 0xFFFFu) : u;
        const f2v x = *(const f2v *)(a.X + (uint64_t)node * d + at_col), h = *(const f2v *)(a.Xhat + (uint64_t)node * d + at_col);
        X[node * 64u + lane] = in ? x : zero;
        Xhat[node * 64u + lane] = in ? h : zero;
    }
    __syncthreads();

    if (wave < TEAMS * CREW) {
        const uint32_t own = ra.batch / CREW;     // the batch is a multiple of 4
        const uint32_t slots = slots_of(groups, NB);
        const auto part = __builtin_amdgcn_make_buffer_rsrc((void *)ra.part, 0, (int)(TEAMS * CREW * 2 * R * 8u * slots), 0x00020000);
        // Cycles from a wave's words to its first request.  us for 200 interactions (89 in the last column) at 0 / 400 / 800 / 1200 /
        // 1600 / 2000 cycles: 8 nodes x 1024, batch 32, H = 2: 344 / 309 / 300 / 302 / 318 / 334, x 4096: 428 / 399 / 387 / 380 / 375 / 385,
        // 12 x 8192, batch 16, H = 3: 481 / 449 / 419 / 409 / 396 / 389, 16 x 936, batch 32, H = 2: 147 / 127 / 121 / 121 / 126 / 131.
        const uint64_t pause = groups == 1 ? 0u : 640u + 24u * groups;
        const float step = ra.lr * ((float)ra.m_rows / (float)ra.batch);
        RunDesc after;                            // the team's next interaction, in vector registers until it is its turn
        auto fetch_after = [&](uint32_t k) {
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            const u4 v = ((SWARM_GLOBAL const u4 *)ra.descs)[min(k, ra.count - 1)];
            after = RunDesc{v.x, v.y, v.z, v.w};
        };
        uint32_t turn = 0;                        // steps this team has taken: numbers the exchanged words
        RunDesc rd = ra.one;
        auto begin = [&](uint32_t k) {            // interaction k of a run: its rows on their way
            rd = RunDesc{first_lane(after.nodes), first_lane(after.event), first_lane(after.flags), first_lane(after.turn)};
            fetch_after(k + TEAMS);
            draw(rd, 0);
            request(0, rows);
            if (((rd.flags >> 8) & 0xFFu) > 1) request(1, rows_ahead);
        };
        if (!single && team < ra.count) {
            fetch_after(team);
            begin(team);
        }
        for (uint32_t k = team, through = 0; k < ra.count; k += TEAMS, ++through) {
            const uint32_t node = rd.nodes & 0xFFFFu, H = (rd.flags >> 8) & 0xFFu;
            wait_for(&finished, rd.turn);         // the initiator's snapshot
            if (lost) break;
            __builtin_amdgcn_s_setprio(2);        // ahead of the teams that wait
            const f2v h = Xhat[node * 64u + lane];
            f2v w = h;
            for (uint32_t q = 0; q < H; ++q) {
                float dots[R];
#pragma unroll
                for (int i = 0; i < R; ++i) dots[i] = fmaf(rows[i].y, w.y, rows[i].x * w.x);
                const float share = wave_totals<R, 32>(dots, lane);      // of row lane / EACH
                const uint32_t tag = ra.tag + turn, set = ((team * 2u + (turn & 1u)) * CREW + mate) * slots * R;
                if (lane % EACH == 0)
                    __hip_atomic_store(ra.part + (set + group * R + lane / EACH), ((unsigned long long)tag << 32) | __float_as_uint(share),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t published = __builtin_readcyclecounter();
                // while the words travel: the rows of the next step, but for the second, which are here
                const float rhs = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (R * (q % EACH) + lane % R)), (int)__float_as_uint(rhs_at)));
                if (q > 0 && q + 1 < H) {
                    if ((q + 1) % EACH == 0) draw(rd, q + 1);
                    request(q + 1, rows_ahead);
                }
                while (__builtin_readcyclecounter() - published < pause) __builtin_amdgcn_s_sleep(1);
                // the residual of row lane % R: the shares of the workgroups lane / R, lane / R + EACH .., in order, then the sum of these
                float residual = 0.f;
                auto collect = [&](auto requests) {   // `requests` words per lane at a time
                    constexpr uint32_t WORDS = decltype(requests)::value;
                    for (uint32_t g0 = 0; g0 < groups && !lost; g0 += WORDS * EACH) {
                        unsigned long long word[WORDS];
                        auto ask = [&](uint32_t i) { word[i] = word_of_agent(part, 8u * lane, 8u * (set + (g0 + i * EACH) * R)); };
                        auto beyond = [&](uint32_t i) { return g0 + i * EACH + lane / R >= groups; };
                        auto missing = [&](uint32_t i) { return !__all((uint32_t)(word[i] >> 32) == tag || beyond(i)); };
                        asm volatile("" ::: "memory");        // not before the pause
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i) ask(i);
                        for (uint64_t since = 0;;) {
                            uint32_t late = 0;
#pragma unroll
                            for (uint32_t i = 0; i < WORDS; ++i) late |= missing(i) ? 1u << i : 0u;
                            if (late == 0) break;
                            if (since == 0) since = wall_clock64();
                            lost = given_up(since);
                            if (lost) break;
                            __builtin_amdgcn_s_sleep(1);
                            asm volatile("" ::: "memory");    // what is read again
#pragma unroll
                            for (uint32_t i = 0; i < WORDS; ++i)
                                if (late & 1u << i) ask(i);
                        }
#pragma unroll
                        for (uint32_t i = 0; i < WORDS; ++i) residual += beyond(i) ? 0.f : __uint_as_float((uint32_t)word[i]);
                    }
                };
                if (groups <= 2 * EACH) collect(std::integral_constant<uint32_t, 2>{});
                else if (groups <= 4 * EACH) collect(std::integral_constant<uint32_t, 4>{});
                else collect(std::integral_constant<uint32_t, 8>{});
                if (lost) break;
                residual = total_from<R>(residual, lane) - rhs;
                f2v even = zero, odd = zero;          // shares of the gradient: two chains of rows per wave
                auto add = [&](int i, f2v &g) {
                    const float r = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residual), i));
                    g.x = fmaf(rows[i].x, r, g.x);
                    g.y = fmaf(rows[i].y, r, g.y);
                };
                if (own == R) {
#pragma unroll
                    for (int i = 0; i < R; i += 2) { add(i, even); add(i + 1, odd); }
                } else {
#pragma unroll
                    for (int i = 0; i < R; i += 2)    // the batch is a multiple of 4, a wave's part of it one of 2
                        if ((uint32_t)i < own) { add(i, even); add(i + 1, odd); }
                }
                // The team's shares meet: a wave's words reach local memory in order.  The set of two steps ago has been read by the mate
                // when its share of the last step is there; the second wave does not wait for that where an interaction ends.
                f2v (*mine)[64] = shares[team][turn & 1u];
                if (mate != 0) wait_for(&arrived[team][0], turn);
                mine[mate][lane] = even + odd;
                ++turn;
                post(&arrived[team][mate], turn);
                if (q + 1 < H || mate == 0) {
                    wait_for(&arrived[team][mate ^ 1u], turn);
                    const f2v g = in ? mine[0][lane] + mine[1][lane] : zero;      // lanes past the row keep a zero
                    w.x = fmaf(-step, g.x, w.x);
                    w.y = fmaf(-step, g.y, w.y);
                }
                if (lost) break;
                if (q + 1 < H) {
#pragma unroll
                    for (int i = 0; i < R; ++i) rows[i] = rows_ahead[i];
                }
            }
            if (lost) break;
            if (mate == 0) {
                if (through) wait_for(&finished, k - TEAMS + 1);     // the one before has been taken
                if (lost) break;
                deltas[team][lane] = w - h;
                post(&stepped[team], through + 1);
                if ((rd.flags & RUN_LAST_LED) && in) *(f2v *)(ra.W + (uint64_t)node * d + col) = w;
            }
            __builtin_amdgcn_s_setprio(0);
            if (k + TEAMS < ra.count) begin(k + TEAMS);
        }
    } else {
        __builtin_amdgcn_s_setprio(3);            // everyone waits for this wave
        uint32_t ri = 0, rj = 0;                  // random words of the pair's rounding
        auto draw = [&](const RunDesc &rd) {
            if constexpr (BITS > 0) {             // a call serves 8 columns: word (column / 2) % 4, low half first
                const Words4 r = stream(here(seed), TAG_SR, 0, lane < 16 ? rd.nodes & 0xFFFFu : rd.nodes >> 16, rd.event, 16u * group + lane % 16u);
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
        RunDesc next = desc(0);
        draw(next);
        uint32_t team = 0, through = 0;
        for (uint32_t k = 0; k < ra.count; ++k) {
            const RunDesc rd = next;
            next = desc(k + 1);
            const uint32_t ni = rd.nodes & 0xFFFFu, nj = rd.nodes >> 16;
            const f2v xi = X[ni * 64u + lane], xj = X[nj * 64u + lane];
            f2v average;
            int zi0 = 0, zi1 = 0, zj0 = 0, zj1 = 0;
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
            if (k + 1 < ra.count) draw(next);
            wait_for(&stepped[team], through + 1);
            if (lost) break;
            const f2v out = average + deltas[team][lane];
            X[ni * 64u + lane] = out;
            Xhat[ni * 64u + lane] = out;
            X[nj * 64u + lane] = average;
            touched[ni] = touched[nj] = 1;
            post(&finished, k + 1);
            if constexpr (BITS > 0) {
                if (rd.flags & RUN_LAST_OF_I) store_code_pair<BITS>(a.ring + (uint64_t)ni * a.row_bytes, col, (uint32_t)zi0, (uint32_t)zi1, in);
                if (rd.flags & RUN_LAST_OF_J) store_code_pair<BITS>(a.ring + (uint64_t)nj * a.row_bytes, col, (uint32_t)zj0, (uint32_t)zj1, in);
            }
            if (++team == TEAMS) { team = 0; ++through; }
        }
    }
    if (lost) {
        __hip_atomic_store(&bail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (lane == 0) atomicOr(&a.counters->barrier_timeouts, 1u);
    }
    if (BITS > 0) report(a.counters, fails, clamped);
    __syncthreads();
    if (bail) return;                             // as far as it got is no state to keep
    for (uint32_t u = wave; u < n; u += RUN_WAVES)
        if (touched[u] != 0 && in) {
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
    if (ra.batch <= 16) lsq_run_kernel<BITS, 16><<<groups, RUN_WAVES * 64, lds, st>>>(ra);
    else lsq_run_kernel<BITS, 32><<<groups, RUN_WAVES * 64, lds, st>>>(ra);
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
