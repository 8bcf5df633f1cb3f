// Local steps of the perceptron objective (see local_mlp.hip for the method) with bf16x3 products: a product a b of float32
// operands is a_lo b_hi + a_hi b_lo + a_hi b_hi on the bf16 matrix cores, accumulated in float32; what is dropped is 2^-16 of it.
// Operands and their layout: mlp_planes.hpp.
//
// Per step and node the weights cross memory once per product and twice per update, which bounds these kernels together with
// the power that matrix cores and local memory draw (2.0 to 2.1 GHz): so the backward product updates W2 with the weights it has
// read, and the update of W1 takes the next step's first product along (mlp_product_kernel with UPDATE), as far as the registers
// hold a gradient's operand.  Features, hidden activations and the logits' gradient are packed by samples (for the products with
// weights) and by columns (for the gradients of the weights), the hidden gradient by columns, all by the kernels that make them.
// us for two steps, against one kernel per product that split both operands on the way into local memory:
//   64 nodes, 1024-4096-1024, batch 128   3576 -> 2979     32 nodes, 800-1504-480, batch 64   454 -> 398, one of them 139 -> 133
//   48 nodes, 1024-4096-1024, batch 64    2244 -> 1897     36 nodes, 608-1280-64, batch 128   347 -> 285, one of them 138 -> 101
//    8 nodes, 1024-4096-1024, batch 32     477 -> 382      64 nodes, 736-1376-896, batch 160  1616 -> 1221, one of them 218 -> 176
//    4 nodes, 1024-2048-512, batch 128     247 -> 196      16 nodes, 800-1504-480, batch 288   653 -> 527, one of them 227 -> 146
// Packing costs where a product is a slab or two deep and its operands are what moves: 31 nodes, 32-96-896, batch 1024 503 -> 527;
// 31 nodes, 608-32-832, batch 32 113 -> 123.
#include <algorithm>
#include <new>
#include <type_traits>

#include "internal.h"
#include "lsq_wave.hpp"
#include "mlp_batch.hpp"
#include "mlp_common.hpp"
#include "mlp_planes.hpp"
#include "objectives.h"

namespace swarm {

enum ProductKind { PRODUCT_HIDDEN = 0, PRODUCT_LOGITS = 1, PRODUCT_BACK = 2 };
constexpr uint32_t MOST_BLOCKS = 5;              // blocks of 32 samples that one workgroup of a product takes at most
constexpr uint32_t MOST_SPLITS = 8;              // of the logits' contraction
// Updates of long batches: fewer tiles of 128 x 128 weights are taken as 64 x 64 (us for two steps, 64 x 64 throughout and this rule:
// 4 nodes, 1024-2048-512, batch 512 386 and 337; 64 nodes, 736-1376-896, batch 192 1858 and 1643; 128 x 128 throughout leaves one
// workgroup to each of 8 nodes, 64-128-32, batch 1024: 178 and 131).
constexpr uint32_t SMALL_TILES = 256;

struct ProductArgs {
    const u4 *act;                  // activations, rows = samples, packed over the contraction index; per slot
    const float *W, *biases;        // models of node 0 whose weights and biases are read, `d` floats per node
    float *W_out;                   // models whose weights (UPDATE) or bias (BACK) take a step
    const uint32_t *nodes;          // slot -> node id, or null for identity
    uint64_t act_stride, d;
    uint64_t weights, bias;         // where in a node's model
    uint32_t ldw, slabs, cols;      // contraction and output columns in blocks of 32
    uint32_t sample_blocks;         // batch / 32
    // workgroups per slot: groups_n of a few column blocks x chunks of samples x splits of the contraction (LOGITS); in all
    uint32_t chunks, splits, groups_n, groups;
    // results
    float *logits;                  // LOGITS: batch x columns per slot, for every split (split_stride floats apart)
    uint64_t split_stride;
    u4 *by_sample, *by_column;      // HIDDEN: activations packed over the columns; HIDDEN, BACK: over the samples
    uint64_t by_sample_stride, by_column_stride;
    uint16_t *mask;                 // HIDDEN writes, BACK reads: bit v of lane l of block (samples, columns): result v is positive
    float *sums;                    // BACK, several chunks: column sums per slot and block of 32 samples, `sums_width` floats each
    uint32_t sums_width;
    // UPDATE: the gradient of the weights is the product of these, packed over the samples
    const u4 *by_row, *own;         // rows: contraction index of the product; its columns
    uint64_t by_row_stride, own_stride;
    float lr;
};

// The three products of half a slab.  TURNED: the operand that is written first in the formula is y.
template <bool TURNED>
__device__ __forceinline__ void add_products(const u4 x_hi, const u4 x_lo, const u4 y_hi, const u4 y_lo, f16v &sum) {
    if (TURNED) {
        sum = mfma(x_hi, y_lo, sum);
        sum = mfma(x_lo, y_hi, sum);
    } else {
        sum = mfma(x_lo, y_hi, sum);
        sum = mfma(x_hi, y_lo, sum);
    }
    sum = mfma(x_hi, y_hi, sum);
}

// Whether a product has the registers to update the weights that it multiplies with.
constexpr bool updates_inside(uint32_t blocks) { return blocks <= 4; }
// Waves of a workgroup: eight where four would leave a compute unit one workgroup for its local memory.
constexpr int product_waves(int blocks, bool update) { return update && blocks == 4 ? 8 : 4; }
// Slabs on their way at a time, as the registers allow: of activations (`per_wave` fragments of each), and of weights.
constexpr int act_depth(int blocks, int per_wave, bool update) {
    if (update) return blocks <= 2 && per_wave <= 2 ? 2 : 1;
    return per_wave <= 2 ? 4 : per_wave <= 4 ? 2 : 1;
}
constexpr int weight_depth(int blocks, bool update) { return update && blocks > 2 ? 2 : 4; }

// result (samples x columns) = activations x weights, and what belongs to it.  RC: a weight row is contiguous along the
// contraction (W[column][k]), else along the columns (W[k][column]).  A wave owns 32 columns and BLOCKS x 32 samples: each
// weight is loaded and split by one wave, once, and the activations' fragments pass through local memory for the waves of a
// workgroup.  The activations are requested before the weights of their turn: loads return in order, and what is needed first
// must not queue behind what may come later.
// UPDATE: the weights of every slab take their step too, before this product (HIDDEN: it belongs to the next step) or after it
// (BACK: it belongs to the same step); the wave's columns of the gradient's second operand stay in registers.
template <int BLOCKS, bool RC, int KIND, bool UPDATE>
__global__ __launch_bounds__(64 * product_waves(BLOCKS, UPDATE), 2) void mlp_product_kernel(const ProductArgs g) {
    constexpr int WAVES = product_waves(BLOCKS, UPDATE), FRAGS = BLOCKS * 4, PER_WAVE = (FRAGS + WAVES - 1) / WAVES;
    constexpr int STAGE = FRAGS * FRAGMENT * (UPDATE ? 2 : 1);
    constexpr int AD = act_depth(BLOCKS, PER_WAVE, UPDATE), WD = weight_depth(BLOCKS, UPDATE);
    constexpr int BOTH = 2;                                                      // chains of dependent products side by side
    constexpr int TILES = KIND == PRODUCT_HIDDEN ? WAVES * 32 * TILE_LD / 4 : 0; // words
    constexpr int ROWS = RC ? WAVES * 512 : 0;                                   // two slabs of weights per wave
    __shared__ u4 lds[2 * STAGE + ROWS > TILES ? 2 * STAGE + ROWS : TILES];
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, r32 = lane & 31u, wave = wave_of_group();
    bool valid;
    const uint32_t q = place_of(blockIdx.x, g.groups, valid);
    if (!valid) return;
    constexpr bool SPLITS = KIND == PRODUCT_LOGITS;
    const uint32_t splits = SPLITS ? g.splits : 1, inner = g.chunks * splits, per_slot = g.groups_n * inner;
    const uint32_t slot = q / per_slot, group = q % per_slot / inner, chunk = q % g.chunks, split = SPLITS ? q % inner / g.chunks : 0;
    const uint32_t node = g.nodes ? g.nodes[slot] : slot, slabs = g.slabs, ldw = g.ldw;
    const uint32_t first_slab = SPLITS ? slabs * split / splits : 0, turns = SPLITS ? slabs * (split + 1) / splits - first_slab : slabs;
    const bool live = group * WAVES + wave < g.cols;
    const uint32_t col = live ? group * WAVES + wave : g.cols - 1;               // of 32 columns
    const u4 *act = g.act + slot * g.act_stride + fragments_at(chunk * BLOCKS, slabs, first_slab);
    const float *W = g.W + node * g.d + g.weights + 32 * first_slab;
    float *Out = UPDATE ? g.W_out + node * g.d + g.weights : nullptr;
    // RC: 8 lanes load a row's 128 bytes, which the wave turns round in local memory (16-byte pieces exchanged by row, so that
    // neither side meets a bank twice); otherwise a lane loads its column's sixteen weights directly.
    const uint32_t weight_bytes = RC ? 4 * ((lane >> 3) * ldw + 4 * (lane & 7u)) : 4 * (4 * half * ldw + r32);
    u4 *const rows = lds + 2 * STAGE + wave * 512;
    const uint32_t put = 8 * (lane >> 3) + ((lane & 7u) ^ (lane >> 4)), turn = (r32 >> 1) & 7u;

    const u4 *by_row = UPDATE ? g.by_row + slot * g.by_row_stride : act;
    struct Staged { u4 act[PER_WAVE], rows[UPDATE ? PER_WAVE : 1]; };
    // Offsets are 32 bits: the slab moves the base, so that one block of samples has no limit (2^20 slabs of 4 KiB are reached by
    // 33.5 M features; several blocks are taken where many workgroups read them, and memory ends long before 2^18 slabs).
    // Blocks past the batch read its last one and are dropped.
    const uint32_t last_block = g.sample_blocks - 1 - chunk * BLOCKS;
    auto load_act = [&](uint32_t t, Staged &r) {
        const Buffer act_buffer = buffer_at(act + (uint64_t)t * 4 * FRAGMENT, ((uint64_t)(BLOCKS - 1) * slabs + 1) * 4096);
        const Buffer rows_buffer = buffer_at(by_row + (uint64_t)t * FRAGS * FRAGMENT, FRAGS * 1024);
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const uint32_t f = wave + WAVES * i;
            if (FRAGS % WAVES == 0 || f < FRAGS) {
                r.act[i] = load16<0>(act_buffer, 16 * lane, (min(f / 4, last_block) * slabs * 4 + f % 4) * 1024);
                if (UPDATE) r.rows[i] = load16<0>(rows_buffer, 16 * lane, f * 1024);
            }
        }
    };
    auto keep_act = [&](u4 *to, const Staged &r) {
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const uint32_t f = wave + WAVES * i;
            if (FRAGS % WAVES == 0 || f < FRAGS) {
                to[f * FRAGMENT + lane] = r.act[i];
                if (UPDATE) to[(FRAGS + f) * FRAGMENT + lane] = r.rows[i];
            }
        }
    };
    auto load_weights = [&](uint32_t t, float w[16]) {
        if (RC) {
            const Buffer b = buffer_at(W + (uint64_t)col * 32 * ldw + 32 * t, 128 * (uint64_t)ldw);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f4 x = __builtin_bit_cast(f4, load16<STREAM>(b, weight_bytes, 32 * i * ldw));
                w[4 * i] = x.x; w[4 * i + 1] = x.y; w[4 * i + 2] = x.z; w[4 * i + 3] = x.w;
            }
        } else {
            // not through a descriptor: its sixteen offsets cost the registers of the pipeline
            SWARM_GLOBAL const float *base = (SWARM_GLOBAL const float *)(W + (uint64_t)t * 32 * ldw + 32 * col);
#pragma unroll
            for (int v = 0; v < 16; ++v) w[v] = __builtin_nontemporal_load(at_bytes(base + row_of(v, 0) * (uint64_t)ldw, weight_bytes));
        }
    };
    auto put_rows = [&](const float w[16], int at) {
#pragma unroll
        for (int i = 0; i < 4; ++i)                // row 8 i + lane / 8: its pieces are exchanged by (row / 2) % 8
            rows[256 * at + 64 * i + (put ^ (4 * (i & 1)))] = __builtin_bit_cast(u4, f4{w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]});
    };
    // piece i of a lane's sixteen weights: by rows of a result (UPDATE) or in the order of a fragment
    auto piece = [&](int i) { return (UPDATE ? 2 * i + half : 4 * (i / 2) + 2 * half + i % 2) ^ turn; };
    auto take_column = [&](float w[16], int at) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f4 x = __builtin_bit_cast(f4, rows[256 * at + 8 * r32 + piece(i)]);
            w[4 * i] = x.x; w[4 * i + 1] = x.y; w[4 * i + 2] = x.z; w[4 * i + 3] = x.w;
        }
    };
    auto split_weights = [&](const float w[16], Halves b[2]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            b[s] = split8(w + 8 * s);
            if (!RC || UPDATE) b[s] = turned(b[s]);
        }
    };

    f16v acc[BLOCKS];
#pragma unroll
    for (int m = 0; m < BLOCKS; ++m) acc[m] = cleared();
    Staged staged[AD];
    u4 own[UPDATE ? FRAGS : 1];
    if (UPDATE) {
        const u4 *at = g.own + slot * g.own_stride + fragments_at(col, BLOCKS, 0);
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) own[UPDATE ? f : 0] = at[f * FRAGMENT + lane];
    }
    float w[WD][16];
    const uint32_t end = turns - 1;
#pragma unroll
    for (int i = 0; i < (AD > WD ? AD : WD); ++i) {
        if (i < AD) load_act(min((uint32_t)i, end), staged[i]);
        if (i < WD) load_weights(min((uint32_t)i, end), w[i]);
    }
    keep_act(lds, staged[0]);
    // RC: slabs of weights pass in pairs, so that a row's 256 bytes are requested together
    auto put_pair = [&](uint32_t t, float (&even)[16], float (&odd)[16]) {      // slabs t and t + 1; the pair WD further on is requested
        put_rows(even, 0);
        put_rows(odd, 1);
        load_weights(min(t + WD, end), even);
        load_weights(min(t + 1 + WD, end), odd);
    };
    if (RC) put_pair(0, w[0], w[1]);
    __syncthreads();
    // Slab t (PHASE = t % 4), after the requests for the slabs after it (past the end: the last one again).  RC: slabs t and, when
    // t is even, t + 1 wait in local memory and the registers hold those after them; otherwise from t on.
    auto slab = [&](uint32_t t, auto phase) {
        constexpr int PHASE = decltype(phase)::value, PARITY = PHASE & 1;
        float (&now)[16] = w[PHASE % WD];
        const u4 *a = lds + PARITY * STAGE;
        float mine[16];
        Halves b[2];
        if (RC) {
            take_column(mine, PARITY);
        } else {
            __builtin_amdgcn_sched_barrier(0);
            if (UPDATE) {
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[v] = now[v];
            }
            split_weights(now, b);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_act(min(t + AD, end), staged[PHASE % AD]);
        if (!RC) load_weights(min(t + WD, end), now);
        else if (!UPDATE && PARITY == 1) put_pair(t + 1, w[(PHASE + 1) % WD], w[(PHASE + 2) % WD]);
        __builtin_amdgcn_sched_barrier(0);          // the requests stay ahead of the work and in this order
        auto update = [&]() {                       // of slab t, in `mine` and in memory
            f16v sum = cleared();
#pragma unroll
            for (int f = 0; f < FRAGS; f += 2)
                add_products<RC>(a[(FRAGS + f) * FRAGMENT + lane], a[(FRAGS + f + 1) * FRAGMENT + lane], own[UPDATE ? f : 0],
                                 own[UPDATE ? f + 1 : 0], sum);
#pragma unroll
            for (int v = 0; v < 16; ++v) mine[v] = fmaf(-g.lr, sum[v], mine[v]);
            if (RC) {                               // back into rows the way they came
                u4 *here = rows + 256 * PARITY, back[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    here[8 * r32 + piece(i)] = __builtin_bit_cast(u4, f4{mine[4 * i], mine[4 * i + 1], mine[4 * i + 2], mine[4 * i + 3]});
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // other lanes' words come next
                const Buffer to = buffer_at(Out + (uint64_t)col * 32 * ldw + 32 * t, 128 * (uint64_t)ldw);
#pragma unroll
                for (int i = 0; i < 4; ++i) back[i] = here[64 * i + (put ^ (4 * (i & 1)))];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // and make room for the next rows
                if (live) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) store16(to, back[i], weight_bytes, 32 * i * ldw);
                }
                if (PARITY == 1) put_pair(t + 1, w[(PHASE + 1) % WD], w[(PHASE + 2) % WD]);
            } else if (live) {
                SWARM_GLOBAL float *to = (SWARM_GLOBAL float *)(Out + (uint64_t)t * 32 * ldw + 32 * col);
#pragma unroll
                for (int v = 0; v < 16; ++v) __builtin_nontemporal_store(mine[v], at_bytes(to + row_of(v, 0) * (uint64_t)ldw, weight_bytes));
            }
        };
        if (UPDATE && RC) update();
        if (RC) split_weights(mine, b);
#pragma unroll
        for (int m = 0; m < BLOCKS; m += BOTH)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                u4 hi[BOTH], lo[BOTH];
#pragma unroll
                for (int i = 0; i < BOTH; ++i)
                    if (m + i < BLOCKS) {
                        hi[i] = a[((m + i) * 4 + 2 * s) * FRAGMENT + lane];
                        lo[i] = a[((m + i) * 4 + 2 * s + 1) * FRAGMENT + lane];
                    }
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int i = 0; i < BOTH; ++i)
                        if (m + i < BLOCKS) acc[m + i] = mfma(p == 0 ? lo[i] : hi[i], p == 1 ? b[s].lo : b[s].hi, acc[m + i]);
            }
        if (UPDATE && !RC) update();
        keep_act(lds + !PARITY * STAGE, staged[(PHASE + 1) % AD]);
        __syncthreads();
    };
    uint32_t t = 0;
    if constexpr (WD == 4) {
        for (; t + 3 < turns; t += 4) {
            slab(t, std::integral_constant<int, 0>{});
            slab(t + 1, std::integral_constant<int, 1>{});
            slab(t + 2, std::integral_constant<int, 2>{});
            slab(t + 3, std::integral_constant<int, 3>{});
        }
        if (t < turns) slab(t, std::integral_constant<int, 0>{});
        if (t + 1 < turns) slab(t + 1, std::integral_constant<int, 1>{});
        if (t + 2 < turns) slab(t + 2, std::integral_constant<int, 2>{});
    } else {
        for (; t + 1 < turns; t += 2) {
            slab(t, std::integral_constant<int, 0>{});
            slab(t + 1, std::integral_constant<int, 1>{});
        }
        if (t < turns) slab(t, std::integral_constant<int, 0>{});
    }
    if (!live) return;

    const uint64_t bias_at = node * g.d + g.bias + 32 * col + r32;
    const float bias = KIND != PRODUCT_BACK && split == 0 ? g.biases[bias_at] : 0.f;
    float column_sum[BLOCKS] = {};                                     // of each block, whatever the chunks: the same bits in all
#pragma unroll
    for (int m = 0; m < BLOCKS; ++m) {
        const uint32_t block = chunk * BLOCKS + m;                     // of 32 samples
        if (block >= g.sample_blocks) break;
        if constexpr (KIND == PRODUCT_LOGITS) {
            float *to = g.logits + split * g.split_stride + ((uint64_t)slot * g.sample_blocks + block) * 32 * (32 * g.cols) + 32 * col;
            const uint32_t lane_bytes = 4 * (4 * half * 32 * g.cols + r32);
#pragma unroll
            for (int v = 0; v < 16; ++v) *at_bytes(uniform(to + (uint64_t)row_of(v, 0) * 32 * g.cols), lane_bytes) = acc[m][v] + bias;
        } else {
            uint16_t *mask = g.mask + (((uint64_t)slot * g.sample_blocks + block) * g.cols + col) * 64 + lane;
            float out[16];
            if constexpr (KIND == PRODUCT_HIDDEN) {
                uint32_t bits = 0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    out[v] = fmaxf(acc[m][v] + bias, 0.f);
                    bits |= (out[v] > 0.f ? 1u : 0u) << v;
                }
                *mask = (uint16_t)bits;
            } else {
                const uint32_t bits = *mask;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    out[v] = (bits >> v) & 1u ? acc[m][v] : 0.f;
                    column_sum[m] += out[v];
                }
            }
            u4 *by_column = g.by_column + slot * g.by_column_stride + fragments_at(col, g.sample_blocks, block);
#pragma unroll
            for (int s = 0; s < 2; ++s) store_fragments(by_column + s * 2 * FRAGMENT, lane, turned(split8(out + 8 * s)));
            if constexpr (KIND == PRODUCT_HIDDEN) {                    // the transpose, through local memory of the wave's own
                float *tile = (float *)lds + wave * 32 * TILE_LD;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                for (int v = 0; v < 16; ++v) tile[row_of(v, half) * TILE_LD + r32] = out[v];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                u4 *by_sample = g.by_sample + slot * g.by_sample_stride + fragments_at(block, g.cols, col);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const f4 x = *(const f4 *)(tile + r32 * TILE_LD + 16 * s + 8 * half), y = *(const f4 *)(tile + r32 * TILE_LD + 16 * s + 8 * half + 4);
                    const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
                    store_fragments(by_sample + s * 2 * FRAGMENT, lane, split8(v));
                }
            }
        }
    }
    if constexpr (KIND == PRODUCT_BACK) {
        float total = 0.f;
#pragma unroll
        for (int m = 0; m < BLOCKS; ++m) {
            const uint32_t block = chunk * BLOCKS + m;
            if (block >= g.sample_blocks) break;
            const float part = column_sum[m] + __shfl_xor(column_sum[m], 32);
            total = m == 0 ? part : total + part;
            if (g.chunks > 1 && half == 0) g.sums[((uint64_t)slot * g.sample_blocks + block) * g.sums_width + 32 * col + r32] = part;
        }
        if (g.chunks == 1 && half == 0) g.W_out[bias_at] = fmaf(-g.lr, total, g.biases[bias_at]);
    }
}

struct UpdateArgs {
    const u4 *a, *b;                // operands, packed over the samples: rows and columns of the weight matrix
    const float *src;               // models, `d` floats per node
    float *dst;
    const uint32_t *nodes;
    uint64_t a_stride, b_stride, d, weights;
    uint32_t ldw, rows, cols, sample_blocks;   // blocks of 32
    uint32_t parts, groups_n, groups;          // a workgroup takes four column blocks and a part of the rows
    float lr;
};

// weights -= lr x (a b^T), the sum over BLOCKS x 32 samples.  A wave owns 32 columns of the matrix, whose operand stays in
// its registers, and goes down the rows in blocks of 32; the rows' operand passes through local memory for the four waves.
template <int BLOCKS>
__global__ __launch_bounds__(256, 2) void mlp_update_kernel(const UpdateArgs g) {
    constexpr int FRAGS = BLOCKS * 4, STAGE = FRAGS * FRAGMENT;
    __shared__ u4 lds[2][STAGE];
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, r32 = lane & 31u, wave = wave_of_group();
    bool valid;
    const uint32_t q = place_of(blockIdx.x, g.groups, valid);
    if (!valid) return;
    const uint32_t per_slot = g.groups_n * g.parts, slot = q / per_slot, part = q % per_slot / g.groups_n, group = q % g.groups_n;
    const uint32_t node = g.nodes ? g.nodes[slot] : slot, ldw = g.ldw;
    const bool live = group * 4 + wave < g.cols;
    const uint32_t col = live ? group * 4 + wave : g.cols - 1;
    const uint32_t first = (uint32_t)((uint64_t)g.rows * part / g.parts), last = (uint32_t)((uint64_t)g.rows * (part + 1) / g.parts);
    const u4 *a = g.a + slot * g.a_stride, *b = g.b + slot * g.b_stride + fragments_at(col, BLOCKS, 0);
    const float *src = g.src + node * g.d + g.weights + 32 * col;
    float *dst = g.dst + node * g.d + g.weights + 32 * col;
    const uint32_t lane_bytes = 4 * (4 * half * ldw + r32);

    auto load_rows = [&](uint32_t r, u4 v[BLOCKS]) {
        const Buffer rows = buffer_at(a + fragments_at(r, BLOCKS, 0), STAGE * 16);
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) v[i] = load16<0>(rows, 16 * lane, (wave + 4 * i) * 1024);
    };
    auto keep_rows = [&](u4 *to, const u4 v[BLOCKS]) {
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) to[(wave + 4 * i) * FRAGMENT + lane] = v[i];
    };
    auto load_weights = [&](uint32_t r, float w[16]) {
        const Buffer from = buffer_at(src + (uint64_t)32 * r * ldw, 128 * (uint64_t)ldw);
#pragma unroll
        for (int v = 0; v < 16; ++v) w[v] = load4(from, lane_bytes, 4 * row_of(v, 0) * ldw);
    };

    u4 columns[FRAGS], staged[2][BLOCKS];
    float w[2][16];
    load_rows(first, staged[0]);
    load_rows(min(first + 1, last - 1), staged[1]);
#pragma unroll
    for (int f = 0; f < FRAGS; ++f) columns[f] = b[f * FRAGMENT + lane];
    load_weights(first, w[0]);
    keep_rows(lds[0], staged[0]);
    __syncthreads();
    // Row block r.  Loads and stores complete in order: what is waited for at the end of a block is better not requested after
    // the block before was stored, hence the second block of operands on its way.
    auto step = [&](uint32_t r, auto parity) {
        constexpr int PARITY = decltype(parity)::value;
        float (&now)[16] = w[PARITY], (&ahead)[16] = w[!PARITY];
        const u4 *rows = lds[PARITY];
        load_rows(min(r + 2, last - 1), staged[PARITY]);
        load_weights(min(r + 1, last - 1), ahead);
        __builtin_amdgcn_sched_barrier(0);
        f16v sum = cleared();
#pragma unroll
        for (int f = 0; f < FRAGS; f += 2)
            add_products<false>(rows[f * FRAGMENT + lane], rows[(f + 1) * FRAGMENT + lane], columns[f], columns[f + 1], sum);
        if (live) {
            const Buffer to = buffer_at(dst + (uint64_t)32 * r * ldw, 128 * (uint64_t)ldw);
#pragma unroll
            for (int v = 0; v < 16; ++v) store4(to, fmaf(-g.lr, sum[v], now[v]), lane_bytes, 4 * row_of(v, 0) * ldw);
        }
        keep_rows(lds[!PARITY], staged[!PARITY]);
        __syncthreads();
    };
    uint32_t r = first;
    for (; r + 1 < last; r += 2) {
        step(r, std::integral_constant<int, 0>{});
        step(r + 1, std::integral_constant<int, 1>{});
    }
    if (r < last) step(r, std::integral_constant<int, 0>{});
}

// The same for any number of samples: a wave takes B x B blocks of 32 x 32 weights, a workgroup of 2 x 2 waves, both operands from
// cache, DEPTH half slabs on their way; the weights are requested behind the first of these.  Bound by the latency of these
// requests until the waves are many, by memory then.  us for two steps, with nothing requested ahead and tiles of 128 x 128, and so:
// 16 nodes, 800-1504-480, batch 288 550 and 528, one of them 280 and 155; 4 nodes, 1024-2048-512, batch 512 393 and 337; 8 nodes,
// 256-512-64, batch 4096 1697 and 755.
template <int B>
__global__ __launch_bounds__(256, 2) void mlp_update_long_kernel(const UpdateArgs g) {
    constexpr int DEPTH = B == 1 ? 4 : 2;
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, r32 = lane & 31u, wave = wave_of_group();
    bool valid;
    const uint32_t q = place_of(blockIdx.x, g.groups, valid);
    if (!valid) return;
    const uint32_t per_slot = g.groups_n * g.parts, slot = q / per_slot, blocks = g.sample_blocks;
    const uint32_t node = g.nodes ? g.nodes[slot] : slot, ldw = g.ldw;
    const uint32_t row0 = q % per_slot / g.groups_n * 2 * B + (wave >> 1) * B, col0 = q % g.groups_n * 2 * B + (wave & 1u) * B;
    if (row0 >= g.rows || col0 >= g.cols) return;
    Buffer a[B], b[B];
#pragma unroll
    for (uint32_t i = 0; i < B; ++i) {
        a[i] = buffer_at(g.a + slot * g.a_stride + fragments_at(min(row0 + i, g.rows - 1), blocks, 0), (uint64_t)blocks * 4096);
        b[i] = buffer_at(g.b + slot * g.b_stride + fragments_at(min(col0 + i, g.cols - 1), blocks, 0), (uint64_t)blocks * 4096);
    }
    const uint64_t from = node * g.d + g.weights + (uint64_t)row0 * 32 * ldw + 32 * col0;
    const uint32_t lane_bytes = 4 * (4 * half * ldw + r32);
    auto inside = [&](uint32_t i, uint32_t j) { return B == 1 || (row0 + i < g.rows && col0 + j < g.cols); };

    f16v sum[B][B];
    float w[B][B][16];
    struct Operands { u4 x[B][2], y[B][2]; } staged[DEPTH];
    const uint32_t halves = 2 * blocks;
    auto load = [&](uint32_t h, Operands &o) {     // half slab h, past the end the last one again
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                o.x[i][p] = load16<0>(a[i], 16 * lane, (2 * min(h, halves - 1) + p) * 1024);
                o.y[i][p] = load16<0>(b[i], 16 * lane, (2 * min(h, halves - 1) + p) * 1024);
            }
    };
#pragma unroll
    for (uint32_t i = 0; i < DEPTH; ++i) load(i, staged[i]);
#pragma unroll
    for (uint32_t i = 0; i < B; ++i)
#pragma unroll
        for (uint32_t j = 0; j < B; ++j) {
            sum[i][j] = cleared();
            if (!inside(i, j)) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                w[i][j][v] = __builtin_nontemporal_load(at_bytes(uniform(g.src + from + (uint64_t)(32 * i + row_of(v, 0)) * ldw + 32 * j), lane_bytes));
        }
    for (uint32_t h = 0; h < halves; h += DEPTH)
#pragma unroll
        for (uint32_t k = 0; k < DEPTH; ++k) {
            if (DEPTH > 2 && h + k >= halves) break;                  // there are two halves to a slab
            const Operands o = staged[k];
            load(h + k + DEPTH, staged[k]);
#pragma unroll
            for (int i = 0; i < B; ++i)
#pragma unroll
                for (int j = 0; j < B; ++j) add_products<false>(o.x[i][0], o.x[i][1], o.y[j][0], o.y[j][1], sum[i][j]);
        }
#pragma unroll
    for (uint32_t i = 0; i < B; ++i)
#pragma unroll
        for (uint32_t j = 0; j < B; ++j) {
            if (!inside(i, j)) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                __builtin_nontemporal_store(fmaf(-g.lr, sum[i][j][v], w[i][j][v]),
                                            at_bytes(uniform(g.dst + from + (uint64_t)(32 * i + row_of(v, 0)) * ldw + 32 * j), lane_bytes));
        }
}

// A minibatch (mlp_batch.hpp), packed.  A workgroup makes up to 128 features (`per_group` times 32) of 32 samples; every thread
// searches the label of its own sample.
constexpr uint32_t BATCH_TILES = 4;
__global__ __launch_bounds__(256) void mlp_packed_batch_kernel(const float *__restrict__ means, const float *__restrict__ cdf,
                                                               const uint32_t *__restrict__ nodes, uint32_t first_node,
                                                               const uint32_t *__restrict__ events,
                                                               uint32_t *__restrict__ labels, u4 *__restrict__ by_sample,
                                                               u4 *__restrict__ by_feature, uint64_t by_sample_stride,
                                                               uint64_t by_feature_stride, uint32_t n_in, uint32_t n_out, uint32_t batch,
                                                               uint32_t per_group, float sigma, uint64_t seed, uint32_t event, uint32_t q) {
    __shared__ __attribute__((aligned(16))) float tiles[BATCH_TILES][32 * TILE_LD];
    const uint32_t slot = blockIdx.z, node = nodes ? nodes[slot] : first_node + slot;
    if (events) event = events[slot];
    const uint32_t row = threadIdx.x >> 3, s = blockIdx.y * 32 + row, at = 4 * (threadIdx.x & 7u);
    const uint32_t first = blockIdx.x * per_group, last = min(first + per_group, n_in / 32);
    const uint32_t y = sample_label(cdf + (uint64_t)node * n_out, n_out, seed, q, node, event, s);
    if (first == 0 && at == 0) labels[(uint64_t)slot * batch + s] = y;
#pragma unroll
    for (uint32_t i = 0; i < BATCH_TILES; ++i) {
        if (first + i >= last) break;
        const uint32_t k = (first + i) * 32 + at;
        *(f4 *)(tiles[i] + row * TILE_LD + at) =
            sample_features(means + (uint64_t)y * n_in + k, sigma, seed, q, node, event, ((uint64_t)s * n_in + k) / 4);
    }
    __syncthreads();
    for (uint32_t i = 0; first + i < last; ++i)
        pack_tile(tiles[i], threadIdx.x, by_sample + slot * by_sample_stride + fragments_at(blockIdx.y, n_in / 32, first + i),
                  by_feature + slot * by_feature_stride + fragments_at(first + i, batch / 32, blockIdx.y));
}

struct SoftmaxArgs {
    const float *logits;            // batch x classes per slot, for every split (split_stride floats apart)
    const uint32_t *labels, *nodes;
    u4 *by_sample, *by_column;      // the gradient, packed
    uint64_t split_stride, by_sample_stride, by_column_stride;
    // its column sums take a step of the bias when the batch is one block of 32 samples, and else go to `sums`
    const float *src;               // models, `d` floats per node
    float *dst, *sums;
    uint64_t d, bias;               // bias: where in a node's model
    uint32_t splits, n_out, batch, sums_width, sums_at;
    float lr;
};

// logits -> (softmax - onehot(y)) / batch, packed, and its column sums.  A workgroup of 16 waves takes 32 rows, a wave two of them;
// 128 columns at a time pass through local memory, every gridDim.z-th 128 in the same workgroup (where there are few
// rows, several workgroups take the same sums, so that more of the chip packs).  Rows of up to 1024 entries stay in registers
// between the passes (maximum, sum of exponentials, result), in groups of 256 that a short row
// leaves out (48 nodes, 32 classes, batch 288: 22.4 -> 16.8 us).  The sums are those of mlp_softmax_grad_kernel (local_mlp.hip) in
// its order: 256 partial sums of every 256th entry, 64 of them by halves at a time, the four results one after the other.
// PER_SIMD: waves per SIMD, four for up to a workgroup per compute unit (73 registers), eight beyond: 31 x 1024 rows of 896
// 87.1 and 75.1 us, 256 x 128 of 1024 99.9 and 84.7; 32 x 64 of 480 10.2 and 11.4, 8 x 32 of 864 9.8 and 11.5.  Exchanges
// through local memory instead of between registers: 85.3, 101.0, 11.2 and 11.2.
template <int PER_SIMD>
__global__ __launch_bounds__(1024, PER_SIMD) void mlp_packed_softmax_grad_kernel(const SoftmaxArgs g) {
    __shared__ __attribute__((aligned(16))) float tiles[2][4][32 * TILE_LD];
    constexpr uint32_t HELD = 16;                  // of 64 entries
    const float *logits = g.logits;
    const uint64_t split_stride = g.split_stride;
    const uint32_t n_out = g.n_out, batch = g.batch, splits = g.splits;
    const uint32_t lane = threadIdx.x & 63u, wave = wave_of_group(), slot = blockIdx.y, node = g.nodes ? g.nodes[slot] : slot;
    const uint32_t blocks = n_out / 32, block = blockIdx.x, sample_blocks = gridDim.x;
    const float inv_b = 1.0f / (float)batch;
    float held[2][HELD], top[2], sum[2];
    uint32_t y[2];
    uint64_t offset[2];
    auto read = [&](int r, uint32_t c) {
        const float *in = logits + offset[r] + c + lane;
        float v = *in;
        for (uint32_t p = 1; p < splits; ++p) v += in[p * split_stride];
        return v;
    };
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint32_t row = block * 32 + 2 * wave + r;
        offset[r] = ((uint64_t)slot * batch + row) * n_out;
        y[r] = g.labels[(uint64_t)slot * batch + row];
    }
    // entries past the row: exp(-inf) = 0.  In fours, of which rows of few classes fill one.
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (uint32_t i = 0; i < HELD; ++i) held[r][i] = -INFINITY;
#pragma unroll
    for (uint32_t four = 0; four < HELD; four += 4)
        if (64 * four < n_out)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (uint32_t i = four; i < four + 4; ++i)
                    if (64 * i + lane < n_out) held[r][i] = logits[offset[r] + 64 * i + lane];
    for (uint32_t p = 1; p < splits; ++p)
#pragma unroll
        for (uint32_t four = 0; four < HELD; four += 4)
            if (64 * four < n_out) {
                float more[2][4];
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i)
                        more[r][i] = 64 * (four + i) + lane < n_out ? logits[offset[r] + p * split_stride + 64 * (four + i) + lane] : 0.f;
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) held[r][four + i] += more[r][i];
            }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float mx = -INFINITY;
#pragma unroll
        for (uint32_t i = 0; i < HELD; ++i) mx = fmaxf(mx, held[r][i]);
        for (uint32_t c = 64 * HELD; c + lane < n_out; c += 64) mx = fmaxf(mx, read(r, c));
        mx = wave_maximum(mx);
        top[r] = mx;
        float part[4] = {};
#pragma unroll
        for (uint32_t four = 0; four < HELD; four += 4)
            if (64 * four < n_out)
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) {
                    held[r][four + i] = expf(held[r][four + i] - mx);
                    part[i] += held[r][four + i];
                }
        for (uint32_t c = 64 * HELD; c < n_out; c += 256)
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i)
                if (c + 64 * i + lane < n_out) part[i] += expf(read(r, c + 64 * i) - mx);
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i] = wave_totals<1, 32>(part + i, lane);
        sum[r] = ((part[0] + part[1]) + part[2]) + part[3];
    }
    uint32_t turn = 0;
    auto result = [&](uint32_t c, const float e[2][2]) {               // columns [c, c + 128), e: the lane's exponentials
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (uint32_t i = 0; i < 2; ++i) {
                const uint32_t col = c + 64 * i + lane;
                if (col < n_out) {
                    const float out = (e[r][i] / sum[r] - (col == y[r] ? 1.f : 0.f)) * inv_b;
                    tiles[turn][2 * i + (lane >> 5)][(2 * wave + r) * TILE_LD + (lane & 31u)] = out;
                }
            }
        __syncthreads();
        const uint32_t mine = wave / 4, column = c / 32 + mine;         // of 32 classes
        if (column < blocks) {
            const float *tile = tiles[turn][mine];
            pack_tile(tile, threadIdx.x & 255u, g.by_sample + slot * g.by_sample_stride + fragments_at(block, blocks, column),
                      g.by_column + slot * g.by_column_stride + fragments_at(column, sample_blocks, block));
            if (wave % 4 == 0) {                  // half a wave's rows one after the other, then the halves
                const float *at = tile + 16 * (lane >> 5) * TILE_LD + (lane & 31u);
                float total = at[0];
#pragma unroll
                for (uint32_t r = 1; r < 16; ++r) total += at[r * TILE_LD];
                total += __shfl_xor(total, 32);
                const uint32_t col = 32 * column + lane;
                if (lane < 32) {
                    if (sample_blocks == 1) g.dst[node * g.d + g.bias + col] = fmaf(-g.lr, total, g.src[node * g.d + g.bias + col]);
                    else g.sums[((uint64_t)slot * sample_blocks + block) * g.sums_width + g.sums_at + col] = total;
                }
            }
        }
        turn ^= 1u;
    };
#pragma unroll
    for (uint32_t i = 0; i < HELD; i += 2)
        if (64 * i < n_out && i / 2 % gridDim.z == blockIdx.z) {
            const float e[2][2] = {{held[0][i], held[0][i + 1]}, {held[1][i], held[1][i + 1]}};
            result(64 * i, e);
        }
    for (uint32_t c = 64 * HELD; c < n_out; c += 128) {
        if (c / 128 % gridDim.z != blockIdx.z) continue;
        float e[2][2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (uint32_t i = 0; i < 2; ++i) e[r][i] = c + 64 * i + lane < n_out ? expf(read(r, c + 64 * i) - top[r]) : 0.f;
        result(c, e);
    }
}

// Biases take a step by the column sums that blocks of 32 samples have left, in the order of the blocks: columns [first, width) of
// the hidden units' sums and, behind them, the classes'.
__global__ __launch_bounds__(256) void mlp_bias_of_blocks_kernel(const float *__restrict__ sums, const float *__restrict__ src,
                                                                 float *__restrict__ dst, const uint32_t *__restrict__ nodes,
                                                                 uint32_t first, uint32_t width, uint32_t n_hid, uint32_t blocks,
                                                                 uint64_t d, uint64_t hidden_off, uint64_t class_off, float lr) {
    const uint32_t slot = blockIdx.y, node = nodes ? nodes[slot] : slot, c = first + blockIdx.x * 256 + threadIdx.x;
    if (c >= width) return;
    sums += (uint64_t)slot * blocks * width + c;
    float sum = sums[0];
#pragma unroll 8
    for (uint32_t k = 1; k < blocks; ++k) sum += sums[(uint64_t)k * width];
    const uint64_t at = (uint64_t)node * d + (c < n_hid ? hidden_off + c : class_off + (c - n_hid));
    dst[at] = fmaf(-lr, sum, src[at]);
}

// How the products of a call are cut.  A workgroup takes `blocks` x 32 samples (as many as fit: every chunk reads the weights
// again) of four or eight blocks of 32 columns.  Where that gives work to no more than half of the compute units, a workgroup takes
// fewer samples (one node of 256, 1024-4096-1024, batch 128, two steps: 560 -> 279 us; 16 nodes of 736-1376-896, batch 160, on the
// line: cut at fewer than 128 workgroups 420, at fewer than 256 469).  The logits' contraction, the longest with the fewest
// columns, is split between workgroups too where the whole swarm leaves compute units without work (4 nodes, 1024-2048-512, batch
// 128: 330 us with neither, 207 so).
// Updates go inside the products where these have enough workgroups, because on their own they are cut by rows too, or where all
// of it is a few slabs.  The lines, inside and apart: batch 32, 512-1024-64, 48 workgroups 103 and 110 us, 1024-4096-1024, 32: 208
// and 193; batch 64, 800-1504-480, 96: 192 and 196, 48: 182 and 166; batch 96, 512-1024-64, 80: 137 and 147; batch 128 (eight waves
// each), 1024-4096-1024, 128: 577 and 575, 96: 546 and 495.  Few slabs, whatever the workgroups: 96-224-64, one node, batch 32 61 and
// 68, batch 96 77 and 80; with the eight waves of batch 128 the other way round (128-512-128 110 and 90, 64-64-128 90 and 78).
// All of it follows from how many nodes step but the splits, which decide the order of the logits' sums and therefore follow from
// the swarm alone; the other choices leave every bit where it is.
struct Plan {
    uint32_t whole, hidden, logits, back;       // blocks
    uint32_t splits;
    bool inside;                                // updates inside the products
};
static Plan plan_of(const MlpObjective &o, uint32_t count) {
    constexpr uint64_t FILL = 256;              // workgroups
    constexpr uint32_t INSIDE[] = {48, 64, 64, 128};        // workgroups from which updates go inside, by blocks
    const uint32_t samples = o.batch / 32;
    Plan p{};
    p.whole = parts_of(samples, parts_of(samples, MOST_BLOCKS));
    auto groups = [](uint32_t columns, uint32_t waves, uint32_t nodes) { return (uint64_t)parts_of(columns / 32, waves) * nodes; };
    auto cut = [&](uint32_t columns, uint32_t splits) {
        uint32_t blocks = p.whole;
        while (blocks > 1 && groups(columns, 4, count) * splits * parts_of(samples, blocks) <= FILL / 2) blocks = (blocks + 1) / 2;
        return blocks;
    };
    p.hidden = cut(o.n_hid, 1);
    p.splits = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({MOST_SPLITS, o.n_hid / 32 / 4, FILL / groups(o.n_out, 4, o.n_nodes)}));
    p.logits = cut(o.n_out, p.splits);
    p.inside = p.whole == samples && updates_inside(samples) &&
               (groups(o.n_hid, product_waves(samples, true), count) >= INSIDE[samples - 1] ||
                (samples < 4 && std::max(o.n_in, o.n_out) <= 128));
    p.back = p.inside ? p.whole : p.hidden;
    return p;
}

// Workspace of the nodes that step together: packed operands, logits for every split, signs of the hidden units, column sums.
struct MlpSplitSpace {
    uint32_t nodes;
    void *own;                                  // what does not fit into the float32 steps' activations
    u4 *x_by_sample, *x_by_feature[2], *hid_by_sample, *hid_by_unit, *dlogits_by_sample, *dlogits_by_class, *dpre_by_unit;
    float *logits, *sums;
    uint16_t *mask;
};

// Where the workspace of s.nodes nodes lies: in x, hid, dhid and dlogits, which hold the float32 steps' activations and which these
// steps do not use otherwise, as far as it fits, the rest from s.own on.  Returns the bytes of the rest.
static uint64_t lay_out(const MlpObjective &o, MlpSplitSpace &s) {
    const uint64_t in = o.n_in, hid = o.n_hid, out = o.n_out, batch = o.batch, value = sizeof(float);
    const Plan all = plan_of(o, o.n_nodes);
    struct Area { uintptr_t at; uint64_t left; };
    Area areas[] = {{(uintptr_t)o.x, value * o.n_nodes * batch * in}, {(uintptr_t)o.hid, value * o.n_nodes * batch * hid},
                    {(uintptr_t)o.dhid, value * o.n_nodes * batch * hid}, {(uintptr_t)o.dlogits, value * o.n_nodes * batch * out}};
    uint64_t rest = 0;
    auto take = [&](auto &p, uint64_t bytes_of_node) {
        const uint64_t bytes = (bytes_of_node * s.nodes + 255) / 256 * 256;
        uintptr_t at = (uintptr_t)s.own + rest;
        bool fits = false;
        for (Area &a : areas) {
            fits = bytes <= a.left;
            if (!fits) continue;
            at = a.at;
            a.at += bytes;
            a.left -= bytes;
            break;
        }
        if (!fits) rest += bytes;
        p = (std::remove_reference_t<decltype(p)>)at;
    };
    take(s.x_by_sample, value * batch * in);             // hi and lo are as large as the value
    take(s.hid_by_sample, value * batch * hid);
    take(s.dpre_by_unit, value * batch * hid);
    take(s.dlogits_by_sample, value * batch * out);
    take(s.hid_by_unit, value * batch * hid);
    take(s.x_by_feature[0], value * batch * in);
    s.x_by_feature[1] = s.x_by_feature[0];
    if (all.inside) take(s.x_by_feature[1], value * batch * in);         // updates inside meet the next step's features
    take(s.dlogits_by_class, value * batch * out);
    take(s.logits, value * all.splits * batch * out);
    if (batch > 32) take(s.sums, value * (batch / 32) * (hid + out));
    take(s.mask, sizeof(uint16_t) * (batch / 32) * (hid / 32) * 64);
    return rest;
}

// For all nodes, or, where memory is short, for as many as find room: the others step after them.
hipError_t alloc_mlp_split(MlpObjective &o) {
    if (o.split) return hipSuccess;
    MlpSplitSpace *s = new (std::nothrow) MlpSplitSpace{};
    if (!s) return hipErrorOutOfMemory;
    hipError_t e = hipErrorOutOfMemory;
    for (uint32_t nodes = o.n_nodes; nodes > 0 && e == hipErrorOutOfMemory; nodes /= 2) {
        s->nodes = nodes;
        const uint64_t bytes = lay_out(o, *s);
        e = bytes > 0 ? hipMalloc(&s->own, bytes) : hipSuccess;
        if (e != hipSuccess) {
            (void)hipGetLastError();                      // reported here, not by the next launch
            s->own = nullptr;
        }
    }
    if (e != hipSuccess) {
        delete s;
        return e;
    }
    (void)lay_out(o, *s);
    o.split = s;
    return hipSuccess;
}

void free_mlp_split(MlpObjective &o) {
    if (!o.split) return;
    if (o.split->own) (void)hipFree(o.split->own);
    delete o.split;
    o.split = nullptr;
}

template <int BLOCKS, bool RC, int KIND, bool UPDATE>
static void product_form(ProductArgs g, uint32_t count, hipStream_t st) {
    constexpr uint32_t WAVES = product_waves(BLOCKS, UPDATE);
    g.groups_n = parts_of(g.cols, WAVES);
    g.groups = g.groups_n * g.chunks * g.splits * count;
    mlp_product_kernel<BLOCKS, RC, KIND, UPDATE><<<whole_turns(g.groups), 64 * WAVES, 0, st>>>(g);
}
template <int BLOCKS>
static void product_kind(const ProductArgs &g, ProductKind kind, bool update, uint32_t count, hipStream_t st) {
    if constexpr (updates_inside(BLOCKS)) {
        if (update && kind == PRODUCT_HIDDEN) return product_form<BLOCKS, true, PRODUCT_HIDDEN, true>(g, count, st);
        if (update) return product_form<BLOCKS, false, PRODUCT_BACK, true>(g, count, st);
    }
    if (kind == PRODUCT_HIDDEN) product_form<BLOCKS, true, PRODUCT_HIDDEN, false>(g, count, st);
    else if (kind == PRODUCT_LOGITS) product_form<BLOCKS, true, PRODUCT_LOGITS, false>(g, count, st);
    else product_form<BLOCKS, false, PRODUCT_BACK, false>(g, count, st);
}
static void launch_product(const ProductArgs &g, ProductKind kind, bool update, uint32_t blocks, uint32_t count, hipStream_t st) {
    switch (blocks) {
        case 1: product_kind<1>(g, kind, update, count, st); break;
        case 2: product_kind<2>(g, kind, update, count, st); break;
        case 3: product_kind<3>(g, kind, update, count, st); break;
        case 4: product_kind<4>(g, kind, update, count, st); break;
        default: product_kind<5>(g, kind, update, count, st); break;
    }
}
static void launch_update(UpdateArgs g, uint32_t count, hipStream_t st) {
    if (g.sample_blocks > MOST_BLOCKS) {
        const bool small = parts_of(g.rows, 4) * parts_of(g.cols, 4) * count < SMALL_TILES;
        g.groups_n = parts_of(g.cols, small ? 2 : 4);
        g.parts = parts_of(g.rows, small ? 2 : 4);
        g.groups = g.groups_n * g.parts * count;
        if (small) mlp_update_long_kernel<1><<<whole_turns(g.groups), 256, 0, st>>>(g);
        else mlp_update_long_kernel<2><<<whole_turns(g.groups), 256, 0, st>>>(g);
        return;
    }
    g.groups_n = parts_of(g.cols, 4);
    g.parts = std::max(1u, std::min(1024 / (count * g.groups_n), g.rows / 2));
    g.groups = g.groups_n * g.parts * count;
    const uint32_t grid = whole_turns(g.groups);
    switch (g.sample_blocks) {
        case 1: mlp_update_kernel<1><<<grid, 256, 0, st>>>(g); break;
        case 2: mlp_update_kernel<2><<<grid, 256, 0, st>>>(g); break;
        case 3: mlp_update_kernel<3><<<grid, 256, 0, st>>>(g); break;
        case 4: mlp_update_kernel<4><<<grid, 256, 0, st>>>(g); break;
        case 5: mlp_update_kernel<5><<<grid, 256, 0, st>>>(g); break;
        default: break;
    }
}

// Steps of up to ws.nodes nodes; base, W: the models of node 0, or of `first_node`, the first slot's, where slots are not named.
static void launch_steps(const float *base, float *W, const MlpObjective &o, const LocalSlots &slots, uint32_t first_node, uint32_t count,
                         uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event, hipStream_t st) {
    const MlpSplitSpace &ws = *o.split;
    const uint32_t *nodes = slots.nodes;
    const uint32_t I = o.n_in, Hd = o.n_hid, O = o.n_out, Bt = o.batch, sb = Bt / 32;
    const uint64_t off_b1 = (uint64_t)Hd * I, off_w2 = off_b1 + Hd, off_b2 = off_w2 + (uint64_t)O * Hd;
    const uint64_t x_s = packed_words(sb, I / 32), x_f = packed_words(I / 32, sb);
    const uint64_t hid_s = packed_words(sb, Hd / 32), hid_u = packed_words(Hd / 32, sb);
    const uint64_t dl_s = packed_words(sb, O / 32), dl_c = packed_words(O / 32, sb), split_stride = (uint64_t)ws.nodes * Bt * O;
    const Plan plan = plan_of(o, count);
    auto product = [&](ProductArgs g, ProductKind kind, bool updating, uint32_t blocks, uint32_t contraction, uint32_t columns) {
        g.slabs = contraction / 32;
        g.cols = columns / 32;
        g.chunks = parts_of(sb, blocks);
        g.splits = kind == PRODUCT_LOGITS ? plan.splits : 1;
        g.split_stride = split_stride;
        launch_product(g, kind, updating, blocks, count, st);
    };
    auto update = [&](UpdateArgs g, uint32_t n_rows, uint32_t n_cols) {
        g.rows = n_rows / 32;
        g.cols = n_cols / 32;
        launch_update(g, count, st);
    };
    auto draw_batch = [&](uint32_t q) {
        // as many features per workgroup as still leave enough workgroups
        const uint32_t tiles = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(BATCH_TILES, (uint64_t)I / 32 * sb * count / 512));
        mlp_packed_batch_kernel<<<dim3(parts_of(I / 32, tiles), sb, count), 256, 0, st>>>(
            o.means, o.cdf, nodes, first_node, slots.events, o.labels, ws.x_by_sample, ws.x_by_feature[q & 1], x_s, x_f, I, O, Bt, tiles, o.data_sigma,
            seed, event, q);
    };
    for (uint32_t q = 0; q < H; ++q) {
        const float *src = q == 0 ? base : W;
        ProductArgs g{};
        g.nodes = nodes; g.W = src; g.biases = src; g.W_out = W; g.d = d; g.sample_blocks = sb; g.mask = ws.mask; g.lr = lr;
        g.by_sample = ws.hid_by_sample; g.by_sample_stride = hid_s;
        // hid = relu(x W1^T + b1)
        ProductArgs first = g;
        first.act = ws.x_by_sample; first.act_stride = x_s;
        first.weights = 0; first.bias = off_b1; first.ldw = I;
        first.by_column = ws.hid_by_unit; first.by_column_stride = hid_u;
        if (q == 0 || !plan.inside) {
            draw_batch(q);
            product(first, PRODUCT_HIDDEN, false, plan.hidden, I, Hd);
        }
        // logits = hid W2^T + b2
        g.act = ws.hid_by_sample; g.act_stride = hid_s;
        g.weights = off_w2; g.bias = off_b2; g.ldw = Hd;
        g.logits = ws.logits;
        product(g, PRODUCT_LOGITS, false, plan.logits, Hd, O);
        const uint32_t share = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(parts_of(O, 128), 256 / ((uint64_t)sb * count)));
        const auto softmax = (uint64_t)sb * count > 256 ? mlp_packed_softmax_grad_kernel<8> : mlp_packed_softmax_grad_kernel<4>;
        softmax<<<dim3(sb, count, share), 1024, 0, st>>>(
            SoftmaxArgs{ws.logits, o.labels, nodes, ws.dlogits_by_sample, ws.dlogits_by_class, split_stride, dl_s, dl_c, src, W, ws.sums, d,
                        off_b2, plan.splits, O, Bt, Hd + O, Hd, lr});
        // dpre = (dlogits W2) * [hid > 0], and b1 <- b1 - eta colsum(dpre) when one chunk is the whole batch (b2 <- b2 - eta colsum(dlogits)
        // went with the softmax when that is one block)
        g.act = ws.dlogits_by_sample; g.act_stride = dl_s;
        g.bias = off_b1; g.sums = ws.sums; g.sums_width = Hd + O;
        g.by_column = ws.dpre_by_unit; g.by_column_stride = hid_u;
        // W2 <- W2 - eta dlogits^T hid
        UpdateArgs u{};
        u.nodes = nodes; u.src = src; u.dst = W; u.d = d; u.sample_blocks = sb; u.lr = lr;
        u.a = ws.dlogits_by_class; u.a_stride = dl_c;
        u.b = ws.hid_by_unit; u.b_stride = hid_u;
        u.weights = off_w2; u.ldw = Hd;
        g.by_row = u.a; g.by_row_stride = u.a_stride; g.own = u.b; g.own_stride = u.b_stride;
        product(g, PRODUCT_BACK, plan.inside, plan.back, O, Hd);
        if (!plan.inside) update(u, O, Hd);
        if (sb > 1) {
            const uint32_t first_sum = plan.back < sb ? 0 : Hd;
            mlp_bias_of_blocks_kernel<<<dim3(parts_of(Hd + O - first_sum, 256), count), 256, 0, st>>>(
                ws.sums, src, W, nodes, first_sum, Hd + O, Hd, sb, d, off_b1, off_b2, lr);
        }
        // W1 <- W1 - eta dpre^T x
        u.a = ws.dpre_by_unit; u.a_stride = hid_u;
        u.b = ws.x_by_feature[q & 1]; u.b_stride = x_f;
        u.weights = 0; u.ldw = I;
        if (!plan.inside || q + 1 == H) {
            update(u, Hd, I);
        } else {
            draw_batch(q + 1);
            first.biases = W;
            first.by_row = u.b; first.by_row_stride = u.b_stride; first.own = u.a; first.own_stride = u.a_stride;
            product(first, PRODUCT_HIDDEN, true, plan.whole, I, Hd);
        }
    }
}

hipError_t launch_local_mlp_split(const float *base, float *W, const MlpObjective &o, const LocalSlots &slots, uint32_t count,
                                  uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event, hipStream_t st) {
    const uint32_t each = parts_of(count, parts_of(count, o.split->nodes));
    for (uint32_t first = 0; first < count; first += each) {
        LocalSlots part;
        if (slots.nodes) part.nodes = slots.nodes + first;
        if (slots.events) part.events = slots.events + first;
        const uint64_t skipped = slots.nodes ? 0 : first * d;
        launch_steps(base + skipped, W + skipped, o, part, first, std::min(each, count - first), d, H, lr, seed, event, st);
    }
    return hipGetLastError();
}

}  // namespace swarm
