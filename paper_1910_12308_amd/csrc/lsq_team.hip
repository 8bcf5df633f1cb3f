// Local SGD steps for least-squares objectives whose swarm has too many columns for a workgroup per slice (local_lsq.hip), by
// teams: the workgroups of a team take one node after the other, each on its own columns, and keep a step's rows of A in
// registers from the residuals to the update, so that these are read once.  Between the two the team's partial residuals are
// added: a workgroup publishes one word per row of the batch, the team's reducing workgroups add these up, in an order that the
// number of columns alone decides, and publish the totals.  While a workgroup waits for them, other teams' workgroups share its
// compute unit; the next step's rows are drawn meanwhile and requested after the update, whose registers they take.
// A word carries the number of the step it belongs to beside the value, so a reader simply waits until the word it needs is there.
// The numbers go on from launch to launch in device memory (a launch in a replayed graph finds fresh ones, too), a copy for each
// workgroup of a team, which it alone reads and moves on: whenever it gets to run, it finds the number of its launch.
// Workgroups wait for one another, so a launch has no more than run at once, and such launches of several swarms on one GPU take
// turns (DeviceTurn).  Where other work keeps some of a team's workgroups from starting all the same, the others' patience ends, 20 ms
// after they began to wait: one of those that hold columns then takes by itself, with the same sums, the nodes whose steps not
// all can finish, and the others end when they have finished theirs (lsq_team_end.hpp).  No wait lasts longer than its patience and two seconds.
#include <algorithm>
#include <mutex>

#include "internal.h"
#include "lsq_team_end.hpp"
#include "lsq_wave.hpp"
#include "objectives.h"
#include "philox.hpp"
#include "uniform_address.hpp"

namespace swarm {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned long long Word;                  // tag << 32 | float bits
constexpr int TEAM_WAVES = 4;
constexpr int TEAM_THREADS = 64 * TEAM_WAVES;
constexpr uint32_t REDUCE_WORDS = 8;              // words a thread of a reducing workgroup asks for at a time
constexpr uint32_t COPIES = 8;                    // of a step's totals, read by every eighth workgroup each: all of them ask for the same lines
constexpr uint32_t WAIT_TICKS = 200000000u;       // 2 s of the 100 MHz wall clock: no wait lasts longer past its patience
// Workgroups that run on a compute unit at once, at most.  The runtime counts vector registers and local memory (seven at a batch of
// 16), not the 800 scalar registers of a SIMD, of which a wave of this kernel takes 112 and 16 for the trap handler: six.  With seven,
// 64 nodes x 131072 columns, batch 16, one step took 24.4 ms, until a workgroup of every team had waited long enough, with six
// 141 us; 100 x 65536 166 and 102, 200 x 16392 52 and 44.
constexpr int TEAM_GROUPS_PER_UNIT = 6;
constexpr unsigned long long MOST_PATIENCE = 1ull << 31;    // both together less than 2^32

// Of a team: the claim of its last launch.
struct LsqTeamHead {
    TeamClaim claim;
    uint32_t pad[30];         // a line each
};

struct LsqTeamArgs {
    const float *base, *A, *b;
    float *W;
    LocalSlots slots;
    LsqTeamHead *heads;
    uint32_t *numbers;        // [team][workgroup] of the next launch's first step
    Word *words, *totals;     // [team][parity; 2: of a workgroup by itself][slice][LSQ_MAX_BATCH], [team][..][COPIES][LSQ_MAX_BATCH]
    float *models;            // [team][d] model of a workgroup by itself between two steps
    DeviceCounters *counters;
    uint64_t d, seed;
    uint32_t patience;        // ticks of the 100 MHz clock
    uint32_t count, teams, slices, reducers, rows_each, H, m_rows, batch, event;
    float lr;
};

struct TeamItem { uint32_t slot, q, H, node, event; };

__device__ __forceinline__ void store_word(SWARM_GLOBAL Word *p, uint32_t tag, float v) {
    __hip_atomic_store(p, ((Word)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ Word load_word(SWARM_GLOBAL const Word *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// ROWS rows of the batch per wave (s = wave ROWS .. wave ROWS + ROWS - 1) of COLS blocks of 256 columns; FULL: the batch has
// 4 ROWS rows.
// Bound by the exchange and memory together: a step of one team is its loads and then about 5 us until the totals are back, hidden
// behind the loads of the other teams on the chip.  Hence as few registers as five workgroups per compute unit take (with four 16 nodes
// x 65544 columns, batch 64, two steps take 140 us instead of 126, with two buffers of rows and three workgroups 154), the first rows
// asked for after the team's number (before, they delay it: 134), totals in copies (one for all: 190).  us for the steps of all nodes
// with 256 rows each, in the wide form (rows read twice, a launch per step or one workgroup per node) and by teams:
//   16 x 65544, batch 64, H = 2    188   122    31 x 16384, batch 32, H = 3   65.9   33.5    64 x 8200, batch 8, H = 2      16.9   13.3
//   64 x 131072, batch 64, H = 1   707   504    64 x 131072, batch 16, H = 1   213    149    16 x 65544, batch 8, H = 2     44.6   25.7
//   9 x 131072, batch 64, H = 4    426   266    64 x 4104, batch 16, H = 1     8.6    8.0    100 x 40000, batch 4, H = 1    32.6   29.9
//   8 x 32768, batch 64, H = 2    46.0  26.5    16 x 16384, batch 16, H = 1    8.1    7.4    40 x 12296, batch 4, H = 2     14.2   11.3
//   100 x 12288, batch 64, H = 2   193   119    33 x 4104, batch 12, H = 2    12.5   10.7    128 x 16392, batch 4, H = 1    17.4   18.1
//   300 x 16384, batch 64, H = 2   993   457                                                 64 x 131072, batch 4, H = 1    59.4   62.8
// (4.4 TB/s of rows read once in the first).  One step of four rows in three rounds or more is the one that loses a little.  Error
// against 64 bits as in the wide form (3.6e-8).
template <int ROWS, int COLS, bool FULL>
__global__ __launch_bounds__(TEAM_THREADS, ROWS <= 4 ? 6 : 5) void lsq_team_kernel(const LsqTeamArgs sa) {
    __shared__ f4 gsum[2][TEAM_WAVES][64 * COLS];
    __shared__ float red[2][TEAM_WAVES][LSQ_MAX_BATCH];
    __shared__ float resid[2][LSQ_MAX_BATCH];
    __shared__ uint32_t rows_of[2][LSQ_MAX_BATCH];
    __shared__ uint32_t quit;                      // the step that was given up, or was not begun
    __shared__ uint32_t ended;                     // and how: TeamWait
    __shared__ TeamClaim head_claim;
    __shared__ uint32_t number;                    // of the launch's first step
    constexpr uint32_t WIDTH = 256 * COLS;
    uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    auto thread = [&] { return 64u * wave + lane; };        // threadIdx.x has no register of its own beside the lane
    auto first = [&] { return wave == 0 && lane == 0; };
    const uint32_t batch = sa.batch, first_row = ROWS * wave, G = sa.slices, all = G + sa.reducers;
    const uint64_t d = sa.d;
    const float step = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(sa.lr * ((float)sa.m_rows / (float)batch))));
    // neighbours of a team on one die: workgroups go round the eight dies
    const uint32_t die = blockIdx.x & 7u, spare = gridDim.x & 7u;
    const uint32_t id = die * (gridDim.x >> 3) + min(die, spare) + (blockIdx.x >> 3);
    const uint32_t team = id / all, member = id - team * all;
    auto find = [&](TeamItem &it, uint32_t slot) {          // the next of the team's slots that takes steps
        for (; slot < sa.count; slot += sa.teams) {
            it.slot = slot; it.q = 0;
            it.H = sa.slots.steps ? sa.slots.steps[slot] : sa.H;
            it.node = sa.slots.nodes ? sa.slots.nodes[slot] : slot;
            it.event = sa.slots.events ? sa.slots.events[slot] : sa.event;
            if (it.H > 0) return true;
        }
        it.slot = slot;
        return false;
    };
    auto advance = [&](TeamItem &it) { return ++it.q < it.H || find(it, it.slot + sa.teams); };
    TeamItem it{};
    if (!find(it, team)) return;
    LsqTeamHead *head = sa.heads + team;
    // A wave that has waited long enough for the step's totals; false: it waits on.
    auto give_up = [&](uint32_t with, bool overdue) {
        uint32_t then = 0;
        if (lane == 0) {
            then = (uint32_t)out_of_patience(
                number, with - number, overdue,
                [&] { return __hip_atomic_load(&head->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                [&](TeamClaim there, TeamClaim mine) { return (TeamClaim)atomicCAS(&head->claim, there, mine); });
            if (then != (uint32_t)TeamWait::GO_ON) {
                quit = with;
                ended = then;
            }
        }
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)then) != (uint32_t)TeamWait::GO_ON;
    };

    auto drawn = [&](const TeamItem &it) {                  // lane s: row s of the batch
        const Words4 r = stream(sa.seed, TAG_BATCH, it.q, it.node, it.event, lane >> 2);
        const uint32_t word = (lane & 3u) == 0 ? r.w0 : (lane & 3u) == 1 ? r.w1 : (lane & 3u) == 2 ? r.w2 : r.w3;
        return scaled_index(word, sa.m_rows);
    };
    // byte offsets into a row's slice, past the row's end those of its last columns
    auto column = [&](uint32_t slice, int c) { return (uint64_t)slice * WIDTH + 256u * c + 4u * lane; };
    auto offset = [&](uint32_t slice, int c) {
        return 4u * (uint32_t)(min(column(slice, c), d - 4) - (uint64_t)slice * WIDTH);
    };
    auto load_model = [&](const float *from, uint32_t slice, f4 w[COLS]) {
        SWARM_GLOBAL const float *p = uniform(from + (uint64_t)slice * WIDTH);
#pragma unroll
        for (int c = 0; c < COLS; ++c) w[c] = *(SWARM_GLOBAL const f4 *)at_bytes(p, offset(slice, c));
    };
    auto store_model = [&](float *p, uint32_t slice, const f4 w[COLS]) {
#pragma unroll
        for (int c = 0; c < COLS; ++c)
            if (wave == (uint32_t)c && column(slice, c) < d) *(f4 *)(p + column(slice, c)) = w[c];
    };
    auto fetch = [&](const TeamItem &it, uint32_t slice, uint32_t rows, f4 a[ROWS][COLS]) {
        const float *An = sa.A + (uint64_t)it.node * sa.m_rows * d + (uint64_t)slice * WIDTH;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {          // past the batch its last row again, which is not used
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)rows, (int)(FULL ? first_row + r : min(first_row + r, batch - 1u)));
            SWARM_GLOBAL const float *p = uniform(An + (uint64_t)row * d);
#pragma unroll
            for (int c = 0; c < COLS; ++c) a[r][c] = *(SWARM_GLOBAL const f4 *)at_bytes(p, offset(slice, c));
        }
    };
    auto offered = [&](uint32_t parity) { return sa.words + ((uint64_t)team * 3 + parity) * G * LSQ_MAX_BATCH; };
    auto summed = [&](uint32_t parity) { return sa.totals + ((uint64_t)team * 3 + parity) * COPIES * LSQ_MAX_BATCH; };
    auto publish = [&](const f4 a[ROWS][COLS], const f4 w[COLS], uint32_t slice, Word *to, uint32_t with) {
        constexpr int PART = ROWS > 8 ? 8 : ROWS, LANES = 64 / PART;          // rows summed together
#pragma unroll
        for (int p = 0; p < ROWS; p += PART) {
            float dots[PART];
#pragma unroll
            for (int r = 0; r < PART; ++r) {
                dots[r] = 0.f;
#pragma unroll
                for (int c = 0; c < COLS; ++c) {
                    const f4 v = a[p + r][c];
                    float acc = v.x * w[c].x;
                    acc = fmaf(v.y, w[c].y, acc); acc = fmaf(v.z, w[c].z, acc); acc = fmaf(v.w, w[c].w, acc);
                    dots[r] += column(slice, c) < d ? acc : 0.f;
                }
            }
            const float total = wave_totals<PART, 32>(dots, lane);           // of row p + lane / LANES
            const uint32_t s = first_row + p + lane / LANES;
            if (lane % LANES == 0 && (FULL || s < batch)) store_word(at_bytes(uniform(to + (uint64_t)slice * LSQ_MAX_BATCH), 8u * s), with, total);
        }
    };
    // The residuals into local memory, by one wave.
    auto wait_total = [&](const Word *from, float b_of_row, uint32_t with, uint32_t parity, uint32_t patience) {     // lane s: the batch's row s
        const uint32_t t0 = (uint32_t)wall_clock64();
        Word word;
        while (true) {
            word = load_word(at_bytes(uniform(from), 8u * min(lane, batch - 1u)));
            if (__all((uint32_t)(word >> 32) == with)) break;
            const uint32_t waited = (uint32_t)wall_clock64() - t0;
            if (waited > patience && give_up(with, waited - patience > WAIT_TICKS)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        resid[parity][lane] = __uint_as_float((uint32_t)word) - b_of_row;
    };
    // rows [j * rows_each, ...) of the batch summed over the slices: a thread takes every (256 / rows_each)-th slice of one row
    auto reduce = [&](uint32_t j, const Word *from, Word *to, uint32_t with, uint32_t parity, uint32_t patience) {
        const uint32_t R = sa.rows_each, row = j * R + (thread() & (R - 1u)), own = min(row, batch - 1u), stride = TEAM_THREADS / R;
        const uint32_t t0 = (uint32_t)wall_clock64();
        float t = 0.f;
        for (uint32_t g0 = thread() / R; __any(g0 < G); g0 += REDUCE_WORDS * stride) {
            Word word[REDUCE_WORDS];
            while (true) {
                bool there = true;
#pragma unroll
                for (uint32_t i = 0; i < REDUCE_WORDS; ++i) word[i] = load_word(at_bytes(uniform(from), 8u * (min(g0 + i * stride, G - 1u) * LSQ_MAX_BATCH + own)));
#pragma unroll
                for (uint32_t i = 0; i < REDUCE_WORDS; ++i) there = there && (uint32_t)(word[i] >> 32) == with;
                if (__all(there)) break;
                if ((uint32_t)wall_clock64() - t0 > patience) {
                    quit = with;                  // and makes no claim
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (uint32_t i = 0; i < REDUCE_WORDS; ++i)
                if (g0 + i * stride < G) t += __uint_as_float((uint32_t)word[i]);
        }
        for (uint32_t off = R; off < 64; off *= 2) t += __shfl_xor(t, off);
        if (lane < R) red[parity][wave][lane] = t;
        __syncthreads();
        if (quit == with) return false;
        if (row < batch) {
            const uint32_t r = thread() & (R - 1u);
            float sum = red[parity][0][r];
#pragma unroll
            for (int w = 1; w < TEAM_WAVES; ++w) sum += red[parity][w][r];
            for (uint32_t copy = thread() / R; copy < COPIES; copy += stride) store_word(at_bytes(uniform(to), 8u * (copy * LSQ_MAX_BATCH + row)), with, sum);
        }
        return true;
    };
    auto update = [&](const f4 a[ROWS][COLS], uint32_t from, uint32_t parity, f4 w[COLS]) {
        const float residuals = resid[from][lane];
        f4 g[COLS];
#pragma unroll
        for (int c = 0; c < COLS; ++c) g[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (FULL || first_row + r < batch) {
                const float rr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residuals), (int)(first_row + r)));
#pragma unroll
                for (int c = 0; c < COLS; ++c) {
                    g[c].x = fmaf(a[r][c].x, rr, g[c].x); g[c].y = fmaf(a[r][c].y, rr, g[c].y);
                    g[c].z = fmaf(a[r][c].z, rr, g[c].z); g[c].w = fmaf(a[r][c].w, rr, g[c].w);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < COLS; ++c) gsum[parity][wave][64 * c + lane] = g[c];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            f4 t = gsum[parity][0][64 * c + lane];
#pragma unroll
            for (int v = 1; v < TEAM_WAVES; ++v) t = t + gsum[parity][v][64 * c + lane];
            w[c].x = fmaf(-step, t.x, w[c].x); w[c].y = fmaf(-step, t.y, w[c].y);
            w[c].z = fmaf(-step, t.z, w[c].z); w[c].w = fmaf(-step, t.w, w[c].w);
        }
    };

    auto base_of = [&](uint32_t node) { return sa.base + (uint64_t)node * d; };
    // Ordinary loads, which a team's workgroups on one die share (past the caches 31 x 16384, batch 16, one step takes 9.7 us instead of
    // 9.2): nobody else moves the number, and a workgroup that misses a claim made just now finds it when it makes its own.
    if (first()) {
        number = sa.numbers[id];
        head_claim = head->claim;
        quit = (uint32_t)(head_claim >> 32) == number ? number : number - 1u;
        ended = (uint32_t)TeamWait::END;
    }
    __syncthreads();
    uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)number);
    auto move_on = [&] {
        if (!first()) return;
        const bool left = quit == tag;
        uint32_t last = tag;                      // past the last step
        if (left) {
            TeamItem rest = it;
            do ++last; while (advance(rest));
        }
        sa.numbers[id] = next_number(number, last - number);
        // All steps are left to all: a claim in every launch, so that none is old enough for the numbers to have come round to it.
        if (!left && member == 0) atomicCAS(&head->claim, head_claim, (TeamClaim)number << 32 | (last - number));
    };
    const bool begun = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(head_claim >> 32)) != tag;     // else the rest has been taken
    if (!begun || member >= G) {
        if (begun)
            do {
                if (!reduce(member - G, offered(tag & 1u), summed(tag & 1u), tag, tag & 1u, sa.patience)) break;
                ++tag;
            } while (advance(it));
        move_on();
        return;
    }
    {
        f4 a[ROWS][COLS], w[COLS];
        float b_of_row;
        auto begin = [&](uint32_t rows) {         // the step's rows on their way
            if (it.q == 0) load_model(base_of(it.node), member, w);
            fetch(it, member, rows, a);
            b_of_row = sa.b[(uint64_t)it.node * sa.m_rows + rows];
        };
        begin(drawn(it));
        while (true) {
            const uint32_t parity = tag & 1u;
            asm volatile("" : "+v"(lane));        // what derives from it is worked out again, or the rows would not fit the registers
            publish(a, w, member, offered(parity), tag);
            TeamItem then = it;
            const bool more = advance(then);
            if (wave == 0) wait_total(summed(parity) + (member % COPIES) * LSQ_MAX_BATCH, b_of_row, tag, parity, sa.patience);
            if (wave == 1 && more) rows_of[parity][lane] = drawn(then);      // the next step's, meanwhile
            __syncthreads();
            if (quit == tag) break;
            const uint32_t rows = rows_of[parity][lane];
            update(a, parity, parity, w);
            asm volatile("" : "+v"(lane));
            if (it.q + 1 == it.H) store_model(sa.W + (uint64_t)it.node * d, member, w);
            ++tag;
            if (!more) break;
            it = then;
            begin(rows);
        }
    }
    move_on();
    if (ended == (uint32_t)TeamWait::LOST && first()) atomicOr(&sa.counters->barrier_timeouts, 1u);
    if (ended == (uint32_t)TeamWait::ALONE) {
        it.q = 0;
        ++tag;                                    // `quit` holds the one that was given up
        uint32_t parity = 0;
        float *own = sa.models + (uint64_t)team * d;
        for (bool more = true; more; more = advance(it), ++tag) {
            f4 a[ROWS][COLS], w[COLS];
            asm volatile("" : "+v"(lane));
            const uint32_t rows = drawn(it);
            const float b_of_row = sa.b[(uint64_t)it.node * sa.m_rows + rows];
            const float *from = it.q ? own : base_of(it.node);
            float *to = it.q + 1 == it.H ? sa.W + (uint64_t)it.node * d : own;
            for (uint32_t g = 0; g < G; ++g) {
                load_model(from, g, w);
                fetch(it, g, rows, a);
                publish(a, w, g, offered(2), tag);
            }
            for (uint32_t j = 0; j < sa.reducers && reduce(j, offered(2), summed(2), tag, parity, WAIT_TICKS); ++j) parity ^= 1u;
            if (wave == 0 && quit != tag) wait_total(summed(2), b_of_row, tag, 0, WAIT_TICKS);
            __syncthreads();
            if (quit == tag) {
                if (first()) atomicOr(&sa.counters->barrier_timeouts, 1u);
                break;
            }
            for (uint32_t g = 0; g < G; ++g, parity ^= 1u) {
                load_model(from, g, w);
                fetch(it, g, rows, a);
                update(a, 0, parity, w);
                store_model(to, g, w);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // the next step reads what other waves have written
            __syncthreads();
        }
    }
}

// Rows of a workgroup: 64 KiB, 32 of batches of at most 16.  More teams than one, and workgroups of several of them on a
// compute unit, keep memory busy while a team waits.
static int team_rows(uint32_t batch) { return batch <= 8 ? 2 : batch <= 16 ? 4 : batch <= 32 ? 8 : 16; }
typedef void (*TeamKernel)(const LsqTeamArgs);
static TeamKernel team_kernel(uint32_t batch) {
    switch (team_rows(batch)) {
        case 2: return batch == 8 ? lsq_team_kernel<2, 4, true> : lsq_team_kernel<2, 4, false>;
        case 4: return batch == 16 ? lsq_team_kernel<4, 2, true> : lsq_team_kernel<4, 2, false>;
        case 8: return batch == 32 ? lsq_team_kernel<8, 2, true> : lsq_team_kernel<8, 2, false>;
        default: return batch == 64 ? lsq_team_kernel<16, 1, true> : lsq_team_kernel<16, 1, false>;
    }
}

// Launches of several swarms on one GPU one after the other: each waits for the last one, where there are several such swarms.  With one
// swarm no launch is recorded, so the GPU is waited for when a second one joins.  Launches captured into a graph take no turns:
// two that run at once may each hold a part of the chip until one of a team's workgroups has waited long enough and takes the rest.
namespace {
struct DeviceTurn {
    std::mutex mutex;
    uint32_t swarms = 0;
    hipEvent_t last = nullptr;                    // there while several swarms are
    bool recorded = false;                        // `last` follows a launch
};
constexpr int MAX_DEVICES = 64;
DeviceTurn device_turns[MAX_DEVICES];
}  // namespace

struct LsqTeams {
    int device;
    uint32_t most, slices, reducers, rows_each;   // most: teams whose workgroups fit the chip together
    LsqTeamHead *heads;
    uint32_t *numbers;
    Word *words, *totals;
    float *models;
};

// o.teams stays null where not even one team fits (at_once: where the chip has no room for all nodes at once), where memory is
// short, or where the runtime cannot tell: the wide form serves.
void alloc_lsq_teams(LsqObjective &o, uint64_t d, uint32_t n, bool at_once) {
    int device = 0, units = 0, each = 0;
    if (hipGetDevice(&device) != hipSuccess || device >= MAX_DEVICES ||
        hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&each, (const void *)team_kernel(o.batch), TEAM_THREADS, 0) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    const uint64_t width = o.batch <= 8 ? 1024 : o.batch <= 32 ? 512 : 256, slices = (d + width - 1) / width;
    uint32_t rows_each = 4;                       // rows a reducing workgroup adds: REDUCE_WORDS words per thread where four rows have no more
    while (rows_each < o.batch && 2 * rows_each * slices <= REDUCE_WORDS * TEAM_THREADS) rows_each *= 2;
    const uint32_t reducers = (o.batch + rows_each - 1) / rows_each;
    const uint64_t most = std::min<uint64_t>((uint64_t)units * std::min(each, TEAM_GROUPS_PER_UNIT) / (slices + reducers), n);
    if (most == 0 || (at_once && most < n)) return;
    LsqTeams t{};
    t.device = device; t.most = (uint32_t)most; t.slices = (uint32_t)slices; t.reducers = reducers; t.rows_each = rows_each;
    const uint64_t head_bytes = sizeof(LsqTeamHead) * most, words = most * 3 * slices * LSQ_MAX_BATCH, totals = most * 3 * COPIES * LSQ_MAX_BATCH;
    const uint64_t exchange = head_bytes + sizeof(Word) * (words + totals), groups = most * (slices + reducers);
    if (hipMalloc((void **)&t.heads, exchange + sizeof(float) * most * d + sizeof(uint32_t) * groups) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    t.words = (Word *)(t.heads + most);
    t.totals = t.words + words;
    t.models = (float *)(t.totals + totals);
    t.numbers = (uint32_t *)(t.models + most * d);
    DeviceTurn &turn = device_turns[device];
    std::lock_guard<std::mutex> lock(turn.mutex);
    // numbers begin at 0 and stay even; no word carries one that is used soon, no claim one at all
    if (hipMemset(t.heads, 0xFF, exchange) != hipSuccess || hipMemset(t.numbers, 0, sizeof(uint32_t) * groups) != hipSuccess ||
        (turn.swarms == 1 &&
         (hipDeviceSynchronize() != hipSuccess || hipEventCreateWithFlags(&turn.last, hipEventDisableTiming) != hipSuccess))) {
        (void)hipGetLastError();
        (void)hipFree(t.heads);
        return;
    }
    turn.swarms += 1;
    o.teams = new LsqTeams(t);
}

void free_lsq_teams(LsqObjective &o) {
    if (!o.teams) return;
    (void)hipFree(o.teams->heads);
    DeviceTurn &turn = device_turns[o.teams->device];
    std::lock_guard<std::mutex> lock(turn.mutex);
    turn.swarms -= 1;
    if (turn.swarms == 1) {
        (void)hipEventDestroy(turn.last);
        turn.last = nullptr; turn.recorded = false;
    }
    delete o.teams;
    o.teams = nullptr;
}

hipError_t launch_lsq_teams(const float *base, float *W, const LsqObjective &o, const LocalSlots &slots, DeviceCounters *counters,
                            uint32_t count, uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event, hipStream_t st) {
    const LsqTeams &t = *o.teams;
    const uint32_t rounds = (count + t.most - 1) / t.most, teams = (count + rounds - 1) / rounds;
    const LsqTeamArgs a{base, o.A, o.b, W, slots, t.heads, t.numbers, t.words, t.totals, t.models, counters, d, seed,
                        (uint32_t)std::min(o.patience, MOST_PATIENCE), count, teams, t.slices, t.reducers, t.rows_each, H, o.m_rows, o.batch, event, lr};
    DeviceTurn &turn = device_turns[t.device];
    std::lock_guard<std::mutex> lock(turn.mutex);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    hipError_t e;
    if (turn.swarms > 1 && (e = hipStreamIsCapturing(st, &capture)) != hipSuccess) return e;
    const bool several = turn.swarms > 1 && capture == hipStreamCaptureStatusNone;
    if (several && turn.recorded && (e = hipStreamWaitEvent(st, turn.last, 0)) != hipSuccess) return e;
    team_kernel(o.batch)<<<teams * (t.slices + t.reducers), TEAM_THREADS, 0, st>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (several) {
        if ((e = hipEventRecord(turn.last, st)) != hipSuccess) return e;
        turn.recorded = true;
    }
    return hipSuccess;
}

}  // namespace swarm
