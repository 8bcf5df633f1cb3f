// Local SGD steps for least-squares node objectives f_i(x) = 1/2 |A_i x - b_i|^2.
// Each step draws `batch` rows uniformly with replacement and uses
//   g~ = (m / batch) A_B^T (A_B w - b_B),
// an unbiased estimate of grad f_i (the paper's requirement on g~_i, Section 2).
// The work per step is two thin matrix-vector products over `batch` rows of A (about one flop per byte).
// Small swarms (at most 256 slices of 512 columns in all, so that the workgroups are resident together) take the
// split form (lsq_split_kernel): one workgroup per slice, which keeps its rows of A in registers for both products
// and its slice of w across all H steps; per step the workgroups of a node exchange only their partial residuals
// (batch floats each) through device memory, each word tagged with the launch and step it belongs to, so a reader
// simply waits until the word it needs carries the right tag (no counters, no fences, nothing to reset).  In a
// batch of Algorithm 1 steps the workgroup then runs the interaction on its slice, which is exactly one gossip tile.
// Of all other swarms, many nodes with few rows take the wide form (lsq_wide_kernel) with one workgroup per node, the rest steps by
// teams of workgroups (lsq_team.hip) or, where not even one node's workgroups fit the chip, the steps update the models themselves
// or their rows are few (one_round_only), the wide form with several per node, which exchange their residuals between launches.
#include <algorithm>
#include <type_traits>

#include "interact_run.hpp"
#include "interact_tile.hpp"
#include "internal.h"
#include "lsq_wave.hpp"
#include "objectives.h"
#include "philox.hpp"

namespace swarm {

// ---- wide form -------------------------------------------------------------------------------------
// Any number of nodes and columns: a node's columns are cut into blocks of 1024 (one float4 per thread), and
// `slices` workgroups of a node share its blocks.  A residual needs the whole row, so a step ends where all of a
// node's workgroups have stored their partial residuals, i.e. at the end of a launch: launch k applies the update of
// step k - 1 to the workgroup's columns and takes the partial residuals of step k on them, H + 1 launches for H
// steps.  With one slice per node (WHOLE) nothing leaves the workgroup and one launch runs all steps, in blocks of 1024
// to 4096 columns.
// Bound by memory: the rows of a step are read twice, once for the residuals and, when these are known, once for the
// update, as they are too many for a workgroup to hold (16 MiB per node at 64 rows of 65536 columns).  16 rows (256 bytes) are in flight
// per thread.  16 nodes x 65544 columns, batch 64, 2 steps: 190 us = 1.07 GB of rows at 5.6 TB/s, against 1.96 ms for
// one workgroup of 1024 threads per node, which left 240 of 256 compute units idle.  Measured without effect: groups
// of nodes whose rows fit the last-level cache (more launches cost more than the hits give), non-temporal loads
// for the second read, the nodes in reverse order in every other launch.
constexpr int WB = 256;                           // threads per workgroup
constexpr uint64_t WIDE_BLOCK = 4 * WB;           // columns a workgroup handles at a time
constexpr uint32_t WIDE_GROUPS = 2048;            // workgroups a launch is cut into where the columns allow it
constexpr uint32_t WIDE_MAX_SLICES = 256;         // every workgroup adds up its node's partial residuals

struct LsqWideArgs {
    const float *base;        // n x d models the steps start from
    float *W;                 // n x d live copies
    const float *A, *b;
    LocalSlots slots;
    float *part;              // [step parity][slot][slice][LSQ_MAX_BATCH] partial residuals
    uint64_t d, seed, part_parity;
    uint32_t H, m_rows, batch, event, slices;
    float lr;
};

template <int THREADS, bool WHOLE>
__global__ __launch_bounds__(THREADS, 4) void lsq_wide_kernel(const LsqWideArgs sa, const uint32_t launch) {
    __shared__ uint32_t rows[2][LSQ_MAX_BATCH];
    __shared__ float resid[LSQ_MAX_BATCH];
    __shared__ float sums[THREADS / 64][LSQ_MAX_BATCH];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, slice = blockIdx.x, slot = blockIdx.y;
    const uint32_t node = sa.slots.nodes ? sa.slots.nodes[slot] : slot;
    const uint32_t H = sa.slots.steps ? sa.slots.steps[slot] : sa.H, event = sa.slots.events ? sa.slots.events[slot] : sa.event;
    if (!WHOLE && launch > H) return;
    constexpr uint64_t BLOCK = 4 * THREADS;
    constexpr int R = 16;                         // rows of A a thread requests at a time
    const uint64_t d = sa.d;
    const float *An = sa.A + (uint64_t)node * sa.m_rows * d, *bn = sa.b + (uint64_t)node * sa.m_rows;
    const float *base = sa.base + (uint64_t)node * d;
    float *wrow = sa.W + (uint64_t)node * d;
    const float step = sa.lr * ((float)sa.m_rows / (float)sa.batch);
    const uint32_t batch = sa.batch;
    const uint64_t own = (d + BLOCK * sa.slices - 1 - BLOCK * slice) / (BLOCK * sa.slices);       // blocks of this slice

    auto draw_rows = [&](uint32_t q) {
        if (threadIdx.x < batch) {
            const Words4 r = stream(sa.seed, TAG_BATCH, q, node, event, threadIdx.x >> 2);
            const uint32_t word = (threadIdx.x & 3u) == 0 ? r.w0 : (threadIdx.x & 3u) == 1 ? r.w1
                                  : (threadIdx.x & 3u) == 2 ? r.w2 : r.w3;
            rows[q & 1u][threadIdx.x] = scaled_index(word, sa.m_rows);
        }
    };
    // this thread's float4 of rows [s0, s0 + R) of step q's batch, issued back to back (a batch is a multiple of 4)
    auto fetch = [&](uint32_t q, uint32_t s0, uint64_t col, f4 a[R]) {
#pragma unroll
        for (int r = 0; r < R; r += 4) {
            if (s0 + r < batch) {
#pragma unroll
                for (int i = r; i < r + 4; ++i) {
                    const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)rows[q & 1u][s0 + i]);
                    a[i] = *(const f4 *)(An + (uint64_t)row * d + col);
                }
            } else {
#pragma unroll
                for (int i = r; i < r + 4; ++i) a[i] = f4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    if (WHOLE && threadIdx.x < LSQ_MAX_BATCH) resid[threadIdx.x] = 0.f;      // stays zero past the batch
    for (uint32_t k = WHOLE ? 0 : launch; k <= (WHOLE ? H : launch); ++k) {       // update of step k - 1, residuals of step k
        const bool update = k > 0, residuals = k < H;
        if (!WHOLE && update) draw_rows(k - 1);
        if (residuals) draw_rows(k);
        if (!WHOLE && update && lane < batch) {
            const float *p = sa.part + (uint64_t)((k - 1) & 1u) * sa.part_parity + (uint64_t)slot * sa.slices * LSQ_MAX_BATCH + lane;
            float t = 0.f;
            for (uint32_t sl = wave; sl < sa.slices; sl += THREADS / 64) t += p[(uint64_t)sl * LSQ_MAX_BATCH];
            sums[wave][lane] = t;
        }
        __syncthreads();
        if (!WHOLE && update) {
            if (threadIdx.x < LSQ_MAX_BATCH) {
                float t = 0.f;
                if (threadIdx.x < batch) {
#pragma unroll
                    for (int w = 0; w < THREADS / 64; ++w) t += sums[w][threadIdx.x];
                    t -= bn[rows[(k - 1) & 1u][threadIdx.x]];
                }
                resid[threadIdx.x] = t;
            }
            __syncthreads();
        }
        const float *src = k <= 1 ? base : wrow;
        if (update) {
            for (uint64_t i = own; i-- > 0;) {    // backwards: the blocks read last are the ones still in cache
                const uint64_t col = (slice + i * sa.slices) * BLOCK + 4ull * threadIdx.x;
                if (col < d) {
                    f4 w = *(const f4 *)(src + col), g = {0.f, 0.f, 0.f, 0.f};
                    for (uint32_t s0 = 0; s0 < batch; s0 += R) {
                        f4 a[R];
                        fetch(k - 1, s0, col, a);
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float rr = resid[s0 + r];           // zero past the batch
                            g.x = fmaf(a[r].x, rr, g.x); g.y = fmaf(a[r].y, rr, g.y);
                            g.z = fmaf(a[r].z, rr, g.z); g.w = fmaf(a[r].w, rr, g.w);
                        }
                    }
                    w.x = fmaf(-step, g.x, w.x); w.y = fmaf(-step, g.y, w.y);
                    w.z = fmaf(-step, g.z, w.z); w.w = fmaf(-step, g.w, w.w);
                    *(f4 *)(wrow + col) = w;
                }
            }
            src = wrow;                           // every thread reads back only what it has written
        }
        if (!residuals) return;
        for (uint32_t s0 = 0; s0 < batch; s0 += R) {
            float acc[R];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = 0.f;
            for (uint64_t i = 0; i < own; ++i) {
                const uint64_t col = (slice + i * sa.slices) * BLOCK + 4ull * threadIdx.x;
                if (col < d) {
                    f4 a[R];
                    fetch(k, s0, col, a);
                    const f4 w = *(const f4 *)(src + col);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        acc[r] = fmaf(a[r].x, w.x, acc[r]); acc[r] = fmaf(a[r].y, w.y, acc[r]);
                        acc[r] = fmaf(a[r].z, w.z, acc[r]); acc[r] = fmaf(a[r].w, w.w, acc[r]);
                    }
                }
            }
            const float total = wave_totals<R>(acc, lane);
            if (lane < R) sums[wave][s0 + lane] = total;
        }
        __syncthreads();
        if (threadIdx.x < batch) {
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < THREADS / 64; ++w) t += sums[w][threadIdx.x];
            if (WHOLE) resid[threadIdx.x] = t - bn[rows[k & 1u][threadIdx.x]];
            else sa.part[(uint64_t)(k & 1u) * sa.part_parity + ((uint64_t)slot * sa.slices + slice) * LSQ_MAX_BATCH + threadIdx.x] = t;
        }
        if (WHOLE) __syncthreads();
    }
}

// ---- wide form, a wave per row -----------------------------------------------------------------------
// One workgroup of 16 waves per node: a wave takes the products with whole rows of the batch, then every thread updates
// float4 columns of its own.  Where it is the better form: lsq_by_rows.
constexpr int ROW_THREADS = 1024;

__global__ __launch_bounds__(ROW_THREADS) void lsq_rows_kernel(const LsqWideArgs sa) {
    __shared__ uint32_t rows[LSQ_MAX_BATCH];
    __shared__ float resid[LSQ_MAX_BATCH];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, slot = blockIdx.x, batch = sa.batch;
    const uint32_t node = sa.slots.nodes ? sa.slots.nodes[slot] : slot;
    const uint32_t H = sa.slots.steps ? sa.slots.steps[slot] : sa.H, event = sa.slots.events ? sa.slots.events[slot] : sa.event;
    const uint64_t d = sa.d;
    const float *An = sa.A + (uint64_t)node * sa.m_rows * d, *bn = sa.b + (uint64_t)node * sa.m_rows;
    float *wrow = sa.W + (uint64_t)node * d;
    const float step = sa.lr * ((float)sa.m_rows / (float)batch);
    for (uint32_t q = 0; q < H; ++q) {
        const float *src = q == 0 ? sa.base + (uint64_t)node * d : wrow;
        if (threadIdx.x < batch) {
            const Words4 r = stream(sa.seed, TAG_BATCH, q, node, event, threadIdx.x >> 2);
            const uint32_t word = (threadIdx.x & 3u) == 0 ? r.w0 : (threadIdx.x & 3u) == 1 ? r.w1
                                  : (threadIdx.x & 3u) == 2 ? r.w2 : r.w3;
            rows[threadIdx.x] = scaled_index(word, sa.m_rows);
        }
        __syncthreads();
        for (uint32_t s = wave; s < batch; s += ROW_THREADS / 64) {
            const float *arow = An + (uint64_t)rows[s] * d;
            float acc = 0.f;
            for (uint64_t k = 4ull * lane; k < d; k += 256) {
                const f4 av = *(const f4 *)(arow + k), wv = *(const f4 *)(src + k);
                acc = fmaf(av.x, wv.x, acc); acc = fmaf(av.y, wv.y, acc);
                acc = fmaf(av.z, wv.z, acc); acc = fmaf(av.w, wv.w, acc);
            }
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            if (lane == 0) resid[s] = acc - bn[rows[s]];
        }
        __syncthreads();
        for (uint64_t k = 4ull * threadIdx.x; k < d; k += 4ull * ROW_THREADS) {
            f4 g = {0.f, 0.f, 0.f, 0.f};
            for (uint32_t s = 0; s < batch; ++s) {
                const f4 av = *(const f4 *)(An + (uint64_t)rows[s] * d + k);
                const float r = resid[s];
                g.x = fmaf(av.x, r, g.x); g.y = fmaf(av.y, r, g.y);
                g.z = fmaf(av.z, r, g.z); g.w = fmaf(av.w, r, g.w);
            }
            f4 wv = *(const f4 *)(src + k);
            wv.x = fmaf(-step, g.x, wv.x); wv.y = fmaf(-step, g.y, wv.y);
            wv.z = fmaf(-step, g.z, wv.z); wv.w = fmaf(-step, g.w, wv.w);
            *(f4 *)(wrow + k) = wv;
        }
        __threadfence_block();
        __syncthreads();
    }
}

// ---- split form ------------------------------------------------------------------------------------
constexpr int SLICE = TILE;                       // columns per workgroup: one gossip tile
constexpr int SW = 4;                             // waves per workgroup
constexpr int RMAX = LSQ_MAX_BATCH / SW;          // rows of the batch a wave holds at most
constexpr uint32_t LSQ_MAX_RESIDENT = 256;        // workgroups of one launch: they wait for one another, so all must
                                                  // be resident at once -- at most one per compute unit
constexpr uint32_t LSQ_MAX_SLICES = LSQ_MAX_RESIDENT / 2;    // a swarm has at least two nodes
constexpr unsigned long long BARRIER_TICKS = 200000000ull;   // 2 s of the 100 MHz wall clock

struct LsqSplitArgs {
    const float *base;        // n x d models the steps start from (plain local steps)
    float *W;                 // n x d live copies
    const float *A, *b;
    LocalSlots slots;         // plain local steps: which nodes
    unsigned long long *part; // exchange: [slot][step parity][slice][LSQ_MAX_BATCH] words (tag << 32 | float bits of
                              // the slice's partial residual); a reader takes a word once it carries this step's tag
    DeviceCounters *counters;
    uint64_t d, seed;
    uint32_t H, m_rows, batch, event, slices;
    uint32_t launch_tag;      // number of this launch << 8: a word's tag is launch_tag | step
    float lr;
};

// Bound by latency: the sums over a wave and the exchange of every step.  A wave sums its rows together (about as many exchanges
// between lanes as rows, without local memory; one by one they were six each) and asks for all words it needs at once (one
// after the other they were a round trip each).  us for the steps of all nodes, with that and before: 8 x 16384, batch 64,
// H = 2: 17.8 and 39.6; 31 x 4096, batch 64, H = 4: 25.7 and 65.2; 8 x 4096, batch 32, H = 2: 10.8 and 18.7; 16 x 4096, batch 16,
// H = 1: 6.5 and 8.1; 8 x 512, batch 4, H = 1: 5.5 and 5.5.  200 interactions of 9 x 4104, batch 64: 1823 and 2565.
// Rows of 4, 16 or 64 of a batch are summed as 1, 4 or 16 per wave: always 16 cost the smallest batches 5 %.
// INTERACT: grid row = one step of Algorithm 1 (descriptor in ia.descs or ia.one): steps from the initiator's snapshot,
// then the interaction on this slice.  Otherwise grid row = one slot of sa.slots, steps from sa.base.
template <int BITS, bool INTERACT>
__global__ __launch_bounds__(SW * 64) void lsq_split_kernel(const LsqSplitArgs sa, const InteractArgs ia) {
    __shared__ uint32_t rows[2][LSQ_MAX_BATCH];
    __shared__ float resid[LSQ_MAX_BATCH];
    __shared__ f4 gsum[SW][SLICE / 4];
    __shared__ float shares[LSQ_MAX_SLICES][LSQ_MAX_BATCH];
    __shared__ int bail;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, slice = blockIdx.x, slot = blockIdx.y;
    SeqDesc sd{};
    uint32_t node, H = sa.H, event = sa.event;
    const float *base = sa.base;
    if (INTERACT) {
        sd = ia.descs ? ia.descs[slot] : ia.one;
        node = sd.ni; H = (sd.flags >> 8) & 0xFFu; event = sd.event;
        base = ia.g.Xhat;
    } else {
        node = sa.slots.nodes ? sa.slots.nodes[slot] : slot;
        if (sa.slots.steps) H = sa.slots.steps[slot];
        if (sa.slots.events) event = sa.slots.events[slot];
    }
    const uint64_t d = sa.d;
    const uint64_t kA = (uint64_t)slice * SLICE + 4ull * lane, kB = kA + SLICE / 2;
    const bool inA = kA < d, inB = kB < d;
    const float *An = sa.A + (uint64_t)node * sa.m_rows * d, *bn = sa.b + (uint64_t)node * sa.m_rows;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const f4 hA = inA ? *(const f4 *)(base + (uint64_t)node * d + kA) : zero;
    const f4 hB = inB ? *(const f4 *)(base + (uint64_t)node * d + kB) : zero;
    f4 wA = hA, wB = hB;
    const float step = sa.lr * ((float)sa.m_rows / (float)sa.batch);
    const uint32_t batch = sa.batch, G = sa.slices, pad_bits = batch <= 16 ? 4 : batch <= 32 ? 5 : 6;
    if (threadIdx.x == 0) bail = 0;

    // rows of step q into rows[q & 1] (threads below batch), then, after a barrier, this wave's rows of the
    // batch (s = wave, wave + 4, ...) into registers: all loads issued back to back
    auto draw_rows = [&](uint32_t q) {
        if (threadIdx.x < batch) {
            const Words4 r = stream(sa.seed, TAG_BATCH, q, node, event, threadIdx.x >> 2);
            const uint32_t word = (threadIdx.x & 3u) == 0 ? r.w0 : (threadIdx.x & 3u) == 1 ? r.w1
                                  : (threadIdx.x & 3u) == 2 ? r.w2 : r.w3;
            rows[q & 1u][threadIdx.x] = scaled_index(word, sa.m_rows);
        }
    };
    auto fetch_rows = [&](uint32_t q, f4 a[RMAX][2]) {
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            const uint32_t s = wave + SW * r;
            a[r][0] = zero; a[r][1] = zero;
            if (s < batch) {
                const float *arow = An + (uint64_t)rows[q & 1u][s] * d;
                if (inA) a[r][0] = *(const f4 *)(arow + kA);
                if (inB) a[r][1] = *(const f4 *)(arow + kB);
            }
        }
    };
    f4 a[RMAX][2], a_next[RMAX][2];
    if (H > 0) {
        draw_rows(0);
        __syncthreads();
        fetch_rows(0, a);
    }
    for (uint32_t q = 0; q < H; ++q) {
        const uint32_t tag = sa.launch_tag | q;
        unsigned long long *mine = sa.part + (((uint64_t)slot * 2 + (q & 1u)) * G + slice) * LSQ_MAX_BATCH;
        auto publish = [&](auto held) {           // the sums of the rows a wave holds, the first `held` of RMAX
            constexpr int ROWS = decltype(held)::value, LANES = 64 / ROWS;
            float dots[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                float acc = 0.f;
                acc = fmaf(a[r][0].x, wA.x, acc); acc = fmaf(a[r][0].y, wA.y, acc);
                acc = fmaf(a[r][0].z, wA.z, acc); acc = fmaf(a[r][0].w, wA.w, acc);
                acc = fmaf(a[r][1].x, wB.x, acc); acc = fmaf(a[r][1].y, wB.y, acc);
                acc = fmaf(a[r][1].z, wB.z, acc); acc = fmaf(a[r][1].w, wB.w, acc);
                dots[r] = acc;
            }
            const float total = wave_totals<ROWS, 32>(dots, lane);           // of row lane / LANES
            const uint32_t s = wave + SW * (lane / LANES);
            if (lane % LANES == 0 && s < batch)
                __hip_atomic_store(mine + s, ((unsigned long long)tag << 32) | __float_as_uint(total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        };
        if (batch <= SW) publish(std::integral_constant<int, 1>{});
        else if (batch <= 4 * SW) publish(std::integral_constant<int, 4>{});
        else publish(std::integral_constant<int, RMAX>{});
        // the next step's rows do not depend on this step's result: request them before waiting
        if (q + 1 < H) {
            draw_rows(q + 1);
            __syncthreads();
            fetch_rows(q + 1, a_next);
        }
        // the residuals: every slice's share, summed in slice order.  A lane asks for up to eight words at once, then again for
        // those that were not there.  The wait is bounded, so that every wave ends whatever happens to the other workgroups.
        {
            const unsigned long long *theirs = sa.part + ((uint64_t)slot * 2 + (q & 1u)) * G * LSQ_MAX_BATCH;
            const unsigned long long t0 = wall_clock64();
            const uint32_t each = 64u >> pad_bits, sidx = lane & ((1u << pad_bits) - 1u);         // slices per wave and request
            const uint32_t g0 = wave * each + (lane >> pad_bits);
            auto collect = [&](auto requests) {
                constexpr int WORDS = decltype(requests)::value;
                for (uint32_t gs = g0; gs - g0 < G; gs += WORDS * SW * each) {
                    unsigned long long word[WORDS];
                    uint32_t late = (1u << WORDS) - 1u;
                    while (true) {
#pragma unroll
                        for (int i = 0; i < WORDS; ++i)
                            if (late & 1u << i) {
                                const uint32_t g = min(gs + i * SW * each, G - 1u);
                                word[i] = __hip_atomic_load(theirs + (uint64_t)g * LSQ_MAX_BATCH + min(sidx, batch - 1u), __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                            }
                        uint32_t still = 0;
#pragma unroll
                        for (int i = 0; i < WORDS; ++i) still |= __all((uint32_t)(word[i] >> 32) == tag) ? 0u : 1u << i;
                        late = still;
                        if (late == 0) break;
                        if (wall_clock64() - t0 > BARRIER_TICKS) { bail = 1; break; }
                        __builtin_amdgcn_s_sleep(1);
                    }
#pragma unroll
                    for (int i = 0; i < WORDS; ++i) {
                        const uint32_t g = gs + i * SW * each;
                        if (g < G && sidx < batch) shares[g][sidx] = __uint_as_float((uint32_t)word[i]);
                    }
                }
            };
            if (G <= SW * each) collect(std::integral_constant<int, 1>{});
            else if (G <= 2 * SW * each) collect(std::integral_constant<int, 2>{});
            else collect(std::integral_constant<int, 8>{});
        }
        __syncthreads();
        if (bail) {
            if (threadIdx.x == 0) atomicOr(&sa.counters->barrier_timeouts, 1u);
            return;
        }
        if (threadIdx.x < batch) {
            float sum = 0.f;
#pragma unroll 8
            for (uint32_t g = 0; g < G; ++g) sum += shares[g][threadIdx.x];
            resid[threadIdx.x] = sum - bn[rows[q & 1u][threadIdx.x]];
        }
        __syncthreads();
        f4 gA = zero, gB = zero;
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            const uint32_t s = wave + SW * r;
            if (s < batch) {
                const float rr = resid[s];
                gA.x = fmaf(a[r][0].x, rr, gA.x); gA.y = fmaf(a[r][0].y, rr, gA.y);
                gA.z = fmaf(a[r][0].z, rr, gA.z); gA.w = fmaf(a[r][0].w, rr, gA.w);
                gB.x = fmaf(a[r][1].x, rr, gB.x); gB.y = fmaf(a[r][1].y, rr, gB.y);
                gB.z = fmaf(a[r][1].z, rr, gB.z); gB.w = fmaf(a[r][1].w, rr, gB.w);
            }
        }
        gsum[wave][lane] = gA;
        gsum[wave][lane + 64] = gB;
        __syncthreads();
        f4 tA = gsum[0][lane], tB = gsum[0][lane + 64];
#pragma unroll
        for (int w = 1; w < SW; ++w) { tA = tA + gsum[w][lane]; tB = tB + gsum[w][lane + 64]; }
        wA.x = fmaf(-step, tA.x, wA.x); wA.y = fmaf(-step, tA.y, wA.y); wA.z = fmaf(-step, tA.z, wA.z); wA.w = fmaf(-step, tA.w, wA.w);
        wB.x = fmaf(-step, tB.x, wB.x); wB.y = fmaf(-step, tB.y, wB.y); wB.z = fmaf(-step, tB.z, wB.z); wB.w = fmaf(-step, tB.w, wB.w);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RMAX; ++r) { a[r][0] = a_next[r][0]; a[r][1] = a_next[r][1]; }
    }
    if (wave != 0) return;
    float *wrow = sa.W + (uint64_t)node * d;
    if (inA) *(f4 *)(wrow + kA) = wA;
    if (inB) *(f4 *)(wrow + kB) = wB;
    if (INTERACT) interact_tile<BITS, 3>(ia, sd, slice, lane, wA - hA, wB - hB);
}

bool lsq_split_fits(uint64_t d, uint32_t n) { return ((d + SLICE - 1) / SLICE) * n <= LSQ_MAX_RESIDENT; }

// Slices per node of the wide form, from the swarm's shape alone: the order in which a node's residuals are summed
// must not depend on how many nodes take steps together (a batch of Algorithm 1 equals its single steps bit for bit).
// One workgroup per node spares the exchange and the launches between steps and is the better form where such workgroups
// keep the chip busy: from 256 nodes on, from 128 up to 16384 columns, from 65 where its blocks of 2048 columns are one
// block or two full ones.  Below, as many slices as make 2048 workgroups, every slice with as many blocks.  us for two
// steps, with slices and with one workgroup:
//   65 x 2048, batch 16     13.0    9.0     128 x 1032, batch 16    13.2    8.4     200 x 4096, batch 16    41.9   29.4
//   80 x 4096, batch 64     64.8   51.6     128 x 4096, batch 64   102.5   64.8     255 x 2048, batch 64   103.7   60.2
//   65 x 3072, batch 64     29.2   43.1     100 x 12288, batch 64  166.5  181.4     200 x 65536, batch 8     233    236
static uint32_t wide_slices(uint64_t d, uint32_t n) {
    if (n >= 256 || (n >= 128 && d <= 16384) || (n > 64 && (d <= 2048 || (d > 3072 && d <= 4096)))) return 1;
    const uint64_t blocks = (d + WIDE_BLOCK - 1) / WIDE_BLOCK;
    const uint64_t most = std::min<uint64_t>({blocks, WIDE_MAX_SLICES, WIDE_GROUPS / n});
    const uint64_t each = (blocks + most - 1) / most;
    return (uint32_t)((blocks + each - 1) / each);
}

// Of the swarms with one workgroup per node, those for which a wave per row is the better form, as measured: a few more
// nodes than compute units, and rows of exactly 16 KiB (their stride matters, not their length: 255 x 4104, batch 16, takes
// 45.0 us with a wave per row and 38.2 in blocks).  us for two steps, a wave per row and blocks of columns:
//   280 x 4096, batch 16   41.5   50.7     300 x 8192, batch 16   91.9  100.2     512 x 4096, batch 16   74.3   81.4
//   300 x 4096, batch 64    167    197     300 x 8192, batch 64    374    380     255 x 4096, batch 64    136    152
//   300 x 5000, batch 16   60.4   55.7     400 x 8192, batch 64    445    433     200 x 4096, batch 64    112    106
static bool lsq_by_rows(uint64_t d, uint32_t n, uint32_t batch) {
    if (n > 256 && n <= 384) return (d > 3072 && d <= 4096) || (d > 6144 && d <= 12288 && batch <= 32);
    return n > 224 && n <= 512 && d == 4096;
}

// Of the swarms that would take one workgroup per node, those whose steps teams take (lsq_team.hip): where a step's rows are many
// enough to outweigh the exchange.  us, one workgroup per node and teams:
//   80 x 4096, batch 64, H = 2    50.5   27.7    200 x 8192, batch 32, H = 2    106   64.5    128 x 8192, batch 16, H = 1    18.5   19.1
//   255 x 2048, batch 64, H = 2   59.1   41.1    300 x 16384, batch 16, H = 1   108   83.3    65 x 2048, batch 16, H = 2      8.8   11.0
//   300 x 4096, batch 64, H = 2    171   81.2    260 x 65536, batch 16, H = 1   489    425    1000 x 2048, batch 16, H = 3    82.3   97.4
//   300 x 16384, batch 64, H = 2   820    338    128 x 16384, batch 64, H = 2   320    152    200 x 4096, batch 16, H = 2    28.2   26.5
static bool teams_pay(uint64_t d, uint32_t batch) {
    return batch >= 64 ? d >= 2048 : batch >= 32 ? d >= 4096 : batch >= 16 && d >= 16384;
}

// Of the swarms whose columns are cut, those with few rows in all whose workgroups of the wide form run at once, four per compute
// unit: teams have to take all their nodes at once there, too, for with their reducing workgroups in a second round they lose more by
// the exchange than they gain by reading rows once.  us, the wide form and teams in two rounds:
//   124 x 8192, batch 4, H = 1     8.7   12.0    100 x 9304, batch 8, H = 1    10.7   13.0    70 x 14336, batch 4, H = 3    25.7   27.3
//   64 x 16384, batch 4, H = 1     9.2   12.0    40 x 25600, batch 8, H = 1    12.7   13.5    16 x 65536, batch 4, H = 1    12.0   12.3
//   64 x 16384, batch 4, H = 2    17.8   19.7    64 x 16384, batch 8, H = 2    26.4   23.8     8 x 131072, batch 4, H = 1   15.7   13.0
static bool one_round_only(uint32_t n, uint32_t slices, uint32_t batch, uint32_t H) {
    return batch <= 8 && batch * H < 16 && slices > 1 && slices <= 32 && n * slices <= 1024;
}

hipError_t alloc_lsq(LsqObjective &o, uint64_t d, uint32_t n, uint32_t H, bool merge_runs) {
    hipError_t e;
    if (!lsq_split_fits(d, n)) {
        o.wide_slices = wide_slices(d, n);
        o.by_rows = o.wide_slices == 1 && lsq_by_rows(d, n, o.batch);
        o.wide_rows = (uint64_t)n * o.wide_slices;
        if ((e = hipMalloc((void **)&o.wide_part, sizeof(float) * 2 * o.wide_rows * LSQ_MAX_BATCH)) != hipSuccess) return e;
        if (o.wide_slices > 1 || teams_pay(d, o.batch)) alloc_lsq_teams(o, d, n, one_round_only(n, o.wide_slices, o.batch, H));
        return hipSuccess;
    }
    const uint64_t slices = (d + SLICE - 1) / SLICE;
    o.part_bytes = sizeof(unsigned long long) * n * 2 * slices * LSQ_MAX_BATCH;
    if ((e = hipMalloc((void **)&o.part, o.part_bytes)) != hipSuccess) return e;
    o.launches = 0;
    if ((e = hipMemset(o.part, 0xFF, o.part_bytes)) != hipSuccess) return e;      // no word carries the tag of a launch yet
    if (!merge_runs) return hipSuccess;
    o.run_part_bytes = lsq_run_bytes(d, o.batch);
    if ((e = hipMalloc((void **)&o.run_part, o.run_part_bytes)) != hipSuccess) return e;
    return hipMemset(o.run_part, 0xFF, o.run_part_bytes);
}

// Launches are numbered so that the words one launch exchanges cannot be taken for another's; when the
// 24-bit number wraps the buffer is wiped (in stream order) before it is reused.
static hipError_t split_args(LsqSplitArgs &sa, const float *base, float *W, LsqObjective &o, const LocalSlots &slots,
                             DeviceCounters *counters, uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event,
                             hipStream_t st) {
    sa = LsqSplitArgs{};
    o.launches = (o.launches + 1) & 0xFFFFFFu;
    if (o.launches == 0xFFFFFFu) {
        const hipError_t e = hipMemsetAsync(o.part, 0xFF, o.part_bytes, st);
        if (e != hipSuccess) return e;
        o.launches = 0;
    }
    sa.launch_tag = o.launches << 8;
    sa.base = base; sa.W = W; sa.A = o.A; sa.b = o.b; sa.slots = slots; sa.part = o.part;
    sa.counters = counters; sa.d = d; sa.seed = seed; sa.H = H; sa.m_rows = o.m_rows; sa.batch = o.batch;
    sa.event = event; sa.slices = (uint32_t)((d + SLICE - 1) / SLICE); sa.lr = lr;
    return hipSuccess;
}

// Threads of the one workgroup per node, where there are far more than compute units: 1024 leave a compute unit one
// workgroup at a time instead of two, so that more of its rows are still in cache for the second read (512 x 2048, batch 16,
// two steps: 38.2 us with 512 threads, 31.2 with 1024; 1000 x 2048, three steps: 89.6 and 68.0).
static void launch_wide(const LsqWideArgs &wa, uint32_t n, uint32_t count, uint32_t max_steps, hipStream_t st) {
    if (wa.slices == 1) {
        const bool one_at_a_time = n >= 500 && wa.d >= 1536 && wa.d <= 3072;
        if (one_at_a_time) lsq_wide_kernel<4 * WB, true><<<dim3(1, count, 1), 4 * WB, 0, st>>>(wa, 0);
        else if (wa.d <= 4 * WB) lsq_wide_kernel<WB, true><<<dim3(1, count, 1), WB, 0, st>>>(wa, 0);
        else if (wa.d <= 64 * WB) lsq_wide_kernel<2 * WB, true><<<dim3(1, count, 1), 2 * WB, 0, st>>>(wa, 0);
        else lsq_wide_kernel<4 * WB, true><<<dim3(1, count, 1), 4 * WB, 0, st>>>(wa, 0);
        return;
    }
    for (uint32_t k = 0; k <= max_steps; ++k) lsq_wide_kernel<WB, false><<<dim3(wa.slices, count, 1), WB, 0, st>>>(wa, k);
}

hipError_t launch_local_lsq(const float *base, float *W, LsqObjective &o, const LocalSlots &slots,
                            DeviceCounters *counters, uint32_t count, uint64_t d, uint32_t H, float lr, uint64_t seed,
                            uint32_t event, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (o.part) {
        LsqSplitArgs sa;
        const hipError_t e = split_args(sa, base, W, o, slots, counters, d, H, lr, seed, event, st);
        if (e != hipSuccess) return e;
        lsq_split_kernel<0, false><<<dim3(sa.slices, count, 1), SW * 64, 0, st>>>(sa, InteractArgs{});
    } else if (o.teams && base != W) {
        return launch_lsq_teams(base, W, o, slots, counters, count, d, H, lr, seed, event, st);
    } else {
        LsqWideArgs wa{base, W, o.A, o.b, slots, o.wide_part, d, seed, o.wide_rows * LSQ_MAX_BATCH,
                       H, o.m_rows, o.batch, event, o.wide_slices, lr};
        if (o.by_rows) lsq_rows_kernel<<<count, ROW_THREADS, 0, st>>>(wa);
        else launch_wide(wa, (uint32_t)(o.wide_rows / o.wide_slices), count, slots.steps ? slots.max_steps : H, st);
    }
    return hipGetLastError();
}

hipError_t launch_lsq_interact(const GossipArgs &g, uint32_t bits, const SeqDesc *descs_dev, const SeqDesc &one, uint32_t count,
                               LsqObjective &o, float lr, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!o.part) return hipErrorInvalidValue;
    LsqSplitArgs sa;
    const hipError_t e = split_args(sa, nullptr, const_cast<float *>(g.W), o, LocalSlots{}, g.counters, g.d, 0, lr, g.seed, 0, st);
    if (e != hipSuccess) return e;
    const InteractArgs ia{g, descs_dev, one, nullptr, nullptr, 0.f, lr};
    const dim3 grid(sa.slices, count, 1);
    switch (bits) {
        case 0: lsq_split_kernel<0, true><<<grid, SW * 64, 0, st>>>(sa, ia); break;
        case 2: lsq_split_kernel<2, true><<<grid, SW * 64, 0, st>>>(sa, ia); break;
        case 4: lsq_split_kernel<4, true><<<grid, SW * 64, 0, st>>>(sa, ia); break;
        case 8: lsq_split_kernel<8, true><<<grid, SW * 64, 0, st>>>(sa, ia); break;
        case 16: lsq_split_kernel<16, true><<<grid, SW * 64, 0, st>>>(sa, ia); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

void free_lsq(LsqObjective &o) {
    if (o.part) (void)hipFree(o.part);
    if (o.run_part) (void)hipFree(o.run_part);
    if (o.wide_part) (void)hipFree(o.wide_part);
    free_lsq_teams(o);
    o = LsqObjective{};
}

}  // namespace swarm
