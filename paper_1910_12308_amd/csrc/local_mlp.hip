// Local SGD steps for the two-layer perceptron objective (in -> hid -> out, ReLU,
// softmax cross-entropy averaged over the batch) on a synthetic Gaussian mixture.
// Every node has its own weights, so each step is a *grouped* problem: one launch per
// GEMM covers all nodes (a one-dimensional grid over (node, tile), numbered so that a node's
// tiles run on one die), each workgroup computing a tile of one node's product (128x128, or smaller: gemm()) on the
// matrix cores (v_mfma_f32_32x32x2f32, float32 in and out).  The same steps from bf16 operands: mlp_split.hip.
//
// Per step:  data (labels, features)  ->  hid = relu(x W1^T + b1)  ->  logits = hid W2^T + b2
//   -> dlogits = (softmax - onehot)/batch -> dpre = (dlogits W2) * [hid > 0]
//   -> W2 -= eta dlogits^T hid, b2 -= eta colsum(dlogits), W1 -= eta dpre^T x, b1 -= eta colsum(dpre).
// The weight updates ride in the two weight-gradient products, so the gradients never reach memory: up to 128 samples
// in mlp_float_update_kernel, which streams down the weight matrix and takes the biases along (at 128 samples the hidden
// bias goes with the epilogue of the backward GEMM, one tile of which holds the whole batch), beyond in the epilogue of
// mlp_gemm_kernel.  Where the logits' product has few tiles it is cut along the hidden units, and the softmax adds the parts.
//
// Tiling: 4 waves per workgroup, each wave a quarter of the tile (64x64 = 2x2 MFMA blocks of 128x128), or 2 waves of a 32x32 block
// each; K is consumed in slabs of 16 staged through LDS (double buffered, the next slab, of small tiles the next four, prefetched
// into registers during the MFMAs).  A 32x32x2 MFMA takes one A and one B value per lane; lanes
// 0-31 carry one k index and lanes 32-63 another, and any pairing is valid as long as A and
// B agree, so lanes 0-31 take k 0..7 of the slab and lanes 32-63 take k 8..15: operands
// whose k runs contiguously in memory are fetched from LDS with two 128-bit reads.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "uniform_address.hpp"
#include "objectives.h"
#include "mlp_batch.hpp"
#include "mlp_common.hpp"
#include "lsq_wave.hpp"

namespace swarm {

constexpr int TK = 16;
constexpr int LDK = TK + 4;      // row length of a [row][k] LDS tile (keeps 16-byte alignment, spreads banks)
constexpr int PAD = 4;           // a row of a [k][row] LDS tile is the tile's rows and this

// Threads of a tile of so many rows: two waves side by side for 32 of them, else two times two.
constexpr int tile_threads(int rows) { return rows == 32 ? 128 : 256; }

enum Epilogue { EPI_BIAS_RELU = 0, EPI_BIAS = 1, EPI_RELU_MASK = 2, EPI_SGD_UPDATE = 3, EPI_PART = 4 };

struct GemmArgs {
    const float *A, *B;          // operand bases
    float *C;                    // output base
    const float *aux;            // bias (per node), ReLU mask source (per slot) or weights to update (per node)
    const uint32_t *nodes;       // slot -> node id, or null for identity
    uint64_t strideA, strideB, strideC, strideAux;   // elements between consecutive nodes / slots
    uint32_t a_by_node, b_by_node, c_by_node, aux_by_node;
    uint32_t M, N, K, lda, ldb, ldc, ldaux;
    float lr;
    // EPI_RELU_MASK only, and only when one tile of 128 rows covers all of them: dst = src - lr * column sums of C, per node
    // (the bias gradient of the hidden layer is the column sum of the matrix this GEMM produces); null = not wanted
    const float *colsum_src;
    float *colsum_dst;
    uint64_t strideColsum;
    // EPI_PART only: the product over K in `parts` pieces of part_k (the last one may be shorter), piece p to C + p * part_stride
    uint32_t parts, part_k;
    uint64_t part_stride;
    uint32_t tiles_n, tiles_m, groups;   // workgroups of the launch: tiles_n x tiles_m (x parts) per slot, total = their product x slots
};

// Which tile a workgroup computes, in the order of the dies (place_of): all tiles of a node on one die, one after the other.
struct Tile { const float *A, *B, *aux, *colsum_src; float *C, *colsum_dst; uint32_t m0, n0, slabs; bool valid; };
template <int EPI, int TM, int TN>
__device__ __forceinline__ Tile tile_of_id(const GemmArgs &g, uint32_t id) {
    Tile t{};
    const uint32_t q = place_of(id, g.groups, t.valid);
    if (!t.valid) return t;
    const uint32_t tiles = g.tiles_n * g.tiles_m, per_slot = EPI == EPI_PART ? tiles * g.parts : tiles, r = q % per_slot % tiles;
    const uint32_t slot = q / per_slot, node = g.nodes ? g.nodes[slot] : slot;
    t.A = g.A + (g.a_by_node ? node : slot) * g.strideA;
    t.B = g.B + (g.b_by_node ? node : slot) * g.strideB;
    t.C = g.C + (g.c_by_node ? node : slot) * g.strideC;
    t.aux = g.aux + (g.aux_by_node ? node : slot) * g.strideAux;
    t.colsum_src = g.colsum_dst ? g.colsum_src + node * g.strideColsum : nullptr;
    t.colsum_dst = g.colsum_dst ? g.colsum_dst + node * g.strideColsum : nullptr;
    t.slabs = g.K / TK;
    if (EPI == EPI_PART) {                       // both operands' k is contiguous
        const uint32_t part = q % per_slot / tiles, k0 = part * g.part_k;
        t.A += k0; t.B += k0; t.C += part * g.part_stride;
        t.slabs = min(g.part_k, g.K - k0) / TK;
    }
    t.m0 = (r / g.tiles_n) * TM;
    t.n0 = (r % g.tiles_n) * TN;
    return t;
}

// Load a ROWS x 16 slab of an operand whose k index is contiguous in memory: P[row * ld + k].
template <int ROWS, int THREADS>
__device__ __forceinline__ void fetch_kc(const float *P, uint32_t ld, uint32_t row0, uint32_t rows, uint32_t k0,
                                         f4 r[ROWS * 4 / THREADS]) {
    const uint32_t t = threadIdx.x;
    SWARM_GLOBAL const float *base = (SWARM_GLOBAL const float *)(P + k0);   // measured: no gain from the marker here
#pragma unroll
    for (int i = 0; i < ROWS * 4 / THREADS; ++i) {
        // rows past the matrix edge re-read its last row: they only feed outputs that are never stored
        const uint32_t row = min(row0 + (t >> 2) + THREADS / 4 * i, rows - 1);
        r[i] = *(SWARM_GLOBAL const f4 *)at_bytes(base, 4 * (row * ld + 4 * (t & 3)));
    }
}
template <int ROWS, int THREADS>
__device__ __forceinline__ void stash_kc(float *lds, const f4 r[ROWS * 4 / THREADS]) {
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < ROWS * 4 / THREADS; ++i) *(f4 *)(lds + ((t >> 2) + THREADS / 4 * i) * LDK + 4 * (t & 3)) = r[i];
}
// Load a 16 x ROWS slab of an operand whose row (m or n) index is contiguous: P[k * ld + row].
// A wave reads 256 / ROWS consecutive k at a time; the part of k that its lanes share makes the base uniform.
template <int ROWS, int THREADS>
__device__ __forceinline__ void fetch_rc(const float *P, uint32_t ld, uint32_t row0, uint32_t rows, uint32_t k0,
                                         uint32_t wave, f4 r[ROWS * 4 / THREADS]) {
    constexpr uint32_t LANES = ROWS / 4, PER_WAVE = 64 / LANES;        // lanes per k, k per wave
    const uint32_t lane = threadIdx.x & 63u, row = min(row0 + 4 * (lane % LANES), rows - 4);
    const uint32_t lane_bytes = 4 * ((lane / LANES) * ld + row);
#pragma unroll
    for (int i = 0; i < ROWS * 4 / THREADS; ++i) {
        SWARM_GLOBAL const float *base = uniform(P + (uint64_t)(k0 + PER_WAVE * wave + THREADS / 64 * PER_WAVE * i) * ld);
        r[i] = *(SWARM_GLOBAL const f4 *)at_bytes(base, lane_bytes);
    }
}
template <int ROWS, int THREADS>
__device__ __forceinline__ void stash_rc(float *lds, const f4 r[ROWS * 4 / THREADS]) {
    constexpr uint32_t LANES = ROWS / 4;
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < ROWS * 4 / THREADS; ++i) *(f4 *)(lds + (t / LANES + THREADS / LANES * i) * (ROWS + PAD) + 4 * (t % LANES)) = r[i];
}

// The 8 operand values of this lane for one 32-row MFMA block: rows row0 + (lane % 32), k run (lane / 32) * 8 .. +7.
template <bool KC, int ROWS>
__device__ __forceinline__ void operand(const float *lds, uint32_t row, uint32_t half, float v[8]) {
    if (KC) {
        const f4 lo = *(const f4 *)(lds + row * LDK + 8 * half), hi = *(const f4 *)(lds + row * LDK + 8 * half + 4);
        v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    } else {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) v[kk] = lds[(8 * half + kk) * (ROWS + PAD) + row];
    }
}

// Epilogues that need a tile of another matrix (the weights to update, the ReLU mask source) request it
// during the K loop, so that its HBM latency hides behind the MFMAs instead of serialising compute phase
// and memory phase.  The values a lane needs (64 in a 128 x 128 tile) are requested in parts, a few after the operand
// fetch of each of the first iterations: loads return in order, so a request for the whole tile ahead
// of the loop would hold back every operand slab behind it until the tile has arrived (and leave memory
// idle for the rest of the loop).  Tiles that lie wholly inside the matrix (all of them when M and N are
// multiples of 128) take straight-line loads and stores; the guarded path serves ragged edges.
struct AuxPos { const float *aux; uint32_t m0, n0, wm, wn, half, r32; bool full_tile; };
// part c = 4 mi + (v / 4): four consecutive rows, all column blocks; 4 MB parts (MB, NB: 32 x 32 blocks of a wave)

// Row group `part` of the lane's values into the registers of row group DEST.  The caller passes
// part == DEST; the addresses are computed from the run-time value, so that they are formed when the
// part is requested (one uniform base, the lane's 32-bit offset, small constants) and not, for all
// values, ahead of the loop that spreads the requests.
template <int EPI, int MB, int NB, int DEST>
__device__ __forceinline__ void prefetch_aux_rows(const GemmArgs &g, const AuxPos p, uint32_t part, float pre[MB][NB][16]) {
    constexpr int mi = DEST >> 2, vq = DEST & 3;
    const uint32_t row0 = p.m0 + p.wm + 32 * (part >> 2) + 8 * (part & 3u);            // uniform
    if (p.full_tile) {
        const uint32_t lane_bytes = 4 * (4 * p.half * g.ldaux + p.r32);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            SWARM_GLOBAL const float *row = uniform(p.aux + (uint64_t)(row0 + j) * g.ldaux + p.n0 + p.wn);
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                SWARM_GLOBAL const float *src = at_bytes(row + 32 * ni, lane_bytes);
                // weights about to be replaced are touched once: keep them out of the way of the cached activations
                pre[mi][ni][4 * vq + j] = EPI == EPI_SGD_UPDATE ? __builtin_nontemporal_load(src) : *src;
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                const uint32_t n = p.n0 + p.wn + 32 * ni + p.r32, m = row0 + 4 * p.half + j;
                pre[mi][ni][4 * vq + j] = (n < g.N && m < g.M) ? p.aux[(uint64_t)m * g.ldaux + n] : 0.f;
            }
    }
}
// The K loops below are unrolled over the parts, so that each part's registers are fixed; the run-time
// copy of the part number keeps the address arithmetic inside the iteration that uses it.
__device__ __forceinline__ uint32_t at_run_time(uint32_t part) {
    asm volatile("" : "+s"(part));
    return part;
}
template <int PART> struct Part { static constexpr int value = PART; };
// Parts [FIRST, 4 MB) for first <= FIRST: what a K loop of `first` iterations has not requested.
template <int EPI, int MB, int NB, int FIRST = 0>
__device__ __forceinline__ void prefetch_aux_rest(const GemmArgs &g, const AuxPos p, uint32_t first, float pre[MB][NB][16]) {
    if (!(EPI == EPI_RELU_MASK || EPI == EPI_SGD_UPDATE)) return;
    if constexpr (FIRST < 4 * MB) {
        if (first <= FIRST) prefetch_aux_rows<EPI, MB, NB, FIRST>(g, p, at_run_time(FIRST), pre);
        prefetch_aux_rest<EPI, MB, NB, FIRST + 1>(g, p, first, pre);
    }
}

// Accumulator layout of a 32x32 block (every 32x32 MFMA shape): register v of lane l holds row
// 8*(v/4) + 4*(l/32) + v%4, column l%32.
// scratch: 64 NB floats of LDS that nothing else uses any more (column sums, when the tile asks for them).
template <int EPI, int MB, int NB>
__device__ __forceinline__ void epilogue(const GemmArgs &g, const Tile &t, f16v acc[MB][NB], uint32_t wm, uint32_t wn,
                                         uint32_t half, uint32_t r32, bool full_tile, float pre[MB][NB][16], float *scratch) {
    constexpr bool SUMS = EPI == EPI_RELU_MASK && MB == 2;       // tiles of 128 rows
    float *C = t.C;
    const float *aux = t.aux;
    const uint32_t m0 = t.m0, n0 = t.n0;
    float colsum[NB] = {};
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) {
            const uint32_t n = n0 + wn + 32 * ni + r32;
            const uint32_t mb = m0 + wm + 32 * mi + 4 * half;
            float bias = 0.f;
            if ((EPI == EPI_BIAS_RELU || EPI == EPI_BIAS) && n < g.N) bias = aux[n];
            float out[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float c = acc[mi][ni][v];
                if (EPI == EPI_BIAS_RELU) c = fmaxf(c + bias, 0.f);
                if (EPI == EPI_BIAS) c = c + bias;
                if (EPI == EPI_RELU_MASK) c = pre[mi][ni][v] > 0.f ? c : 0.f;
                if (EPI == EPI_SGD_UPDATE) c = fmaf(-g.lr, c, pre[mi][ni][v]);
                out[v] = c;
                if (SUMS && (full_tile || mb + 8 * (v >> 2) + (v & 3) < g.M)) colsum[ni] += c;
            }
            if (full_tile) {
                const uint32_t lane_bytes = 4 * (4 * half * g.ldc + r32);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    SWARM_GLOBAL float *row =
                        uniform(C + (uint64_t)(m0 + wm + 32 * mi + 8 * (v >> 2) + (v & 3)) * g.ldc + n0 + wn + 32 * ni);
                    SWARM_GLOBAL float *dst = at_bytes(row, lane_bytes);
                    if (EPI == EPI_SGD_UPDATE) __builtin_nontemporal_store(out[v], dst); else *dst = out[v];
                }
            } else if (n < g.N) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t m = mb + 8 * (v >> 2) + (v & 3);
                    if (m < g.M) C[(uint64_t)m * g.ldc + n] = out[v];
                }
            }
        }
    if (SUMS && t.colsum_dst) {                          // uniform: every wave of the workgroup takes this path
        // a column's rows sit in the two halves of a wave and in the two waves with the same wn
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) colsum[ni] += __shfl_xor(colsum[ni], 32);
        if (wm != 0 && half == 0) {
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) scratch[wn + 32 * ni + r32] = colsum[ni];
        }
        __syncthreads();
        if (wm == 0 && half == 0) {
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                const uint32_t n = n0 + wn + 32 * ni + r32;
                if (n < g.N) t.colsum_dst[n] = fmaf(-g.lr, colsum[ni] + scratch[wn + 32 * ni + r32], t.colsum_src[n]);
            }
        }
    }
}

// C (M x N) = op(A) op(B) with A_KC: A stored [m][k] else [k][m]; B_KC: B stored [n][k] else [k][n].
template <bool A_KC, bool B_KC, int EPI, int TM, int TN>
__global__ __launch_bounds__(tile_threads(TM), TM * TN > 64 * 64 ? 2 : 4) void mlp_gemm_kernel(const GemmArgs g) {
    constexpr int THREADS = tile_threads(TM), WAVES_M = THREADS / 128;
    constexpr int MB = TM / (32 * WAVES_M), NB = TN / 64, PARTS = 4 * MB;
    constexpr int A_TILE = A_KC ? TM * LDK : TK * (TM + PAD), B_TILE = B_KC ? TN * LDK : TK * (TN + PAD);
    __shared__ __attribute__((aligned(16))) float lds_a[2][A_TILE];
    __shared__ __attribute__((aligned(16))) float lds_b[2][B_TILE];
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, r32 = lane & 31u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // scalar: bases stay uniform
    const uint32_t wm = (wave >> 1) * (TM / WAVES_M), wn = (wave & 1u) * (TN / 2);
    // Slabs on their way to local memory.  A wave of a 64 x 64 tile is through a slab in 500 cycles, a quarter of what one takes to
    // arrive: with one slab ahead 8 nodes, 1024-4096-1024, batch 32 take 499 us for two steps instead of 463, 50 nodes, 800-1504-480,
    // batch 64 764 instead of 744, launches of a few slabs the same.
    constexpr int AHEAD = TM * TN <= 64 * 64 ? 4 : 1;

    constexpr int FA = TM * 4 / THREADS, FB = TN * 4 / THREADS;         // float4 of a slab per thread
    f4 ring_a[AHEAD][FA], ring_b[AHEAD][FB];
    auto fetch = [&](const Tile &t, uint32_t k0, f4 (&ra)[FA], f4 (&rb)[FB]) {
        if (A_KC) fetch_kc<TM, THREADS>(t.A, g.lda, t.m0, g.M, k0, ra); else fetch_rc<TM, THREADS>(t.A, g.lda, t.m0, g.M, k0, wave, ra);
        if (B_KC) fetch_kc<TN, THREADS>(t.B, g.ldb, t.n0, g.N, k0, rb); else fetch_rc<TN, THREADS>(t.B, g.ldb, t.n0, g.N, k0, wave, rb);
    };
    auto stash = [&](int buf, const f4 (&ra)[FA], const f4 (&rb)[FB]) {
        if (A_KC) stash_kc<TM, THREADS>(lds_a[buf], ra); else stash_rc<TM, THREADS>(lds_a[buf], ra);
        if (B_KC) stash_kc<TN, THREADS>(lds_b[buf], rb); else stash_rc<TN, THREADS>(lds_b[buf], rb);
    };

    const Tile t = tile_of_id<EPI, TM, TN>(g, blockIdx.x);
    if (!t.valid) return;
    const uint32_t slabs = t.slabs;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(t, min((uint32_t)i, slabs - 1) * TK, ring_a[i], ring_b[i]);
    f16v acc[MB][NB];
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    const bool full_tile = t.m0 + TM <= g.M && t.n0 + TN <= g.N;
    float pre[MB][NB][16];
    const AuxPos aux_pos{t.aux, t.m0, t.n0, wm, wn, half, r32, full_tile};

    stash(0, ring_a[0], ring_b[0]);
    __syncthreads();
    // iteration s of the K loop (s % 8 == TURN); the first ones also request two parts of the other tile each,
    // which leaves the rest of even the shortest K loop (K = 128: eight iterations) to cover their latency
    auto iteration = [&](uint32_t s, auto turn) {
        constexpr int TURN = decltype(turn)::value, cur = TURN & 1;
        constexpr int FREE = TURN % AHEAD, NEXT = (TURN + 1) % AHEAD;
        if constexpr (AHEAD > 1) fetch(t, min(s + AHEAD, slabs - 1) * TK, ring_a[FREE], ring_b[FREE]);     // no branch: what is on its way stays countable
        else if (s + 1 < slabs) fetch(t, (s + 1) * TK, ring_a[0], ring_b[0]);
        if constexpr ((EPI == EPI_RELU_MASK || EPI == EPI_SGD_UPDATE) && 2 * TURN + 1 < PARTS)
            if (s < PARTS / 2) {
                prefetch_aux_rows<EPI, MB, NB, 2 * TURN>(g, aux_pos, at_run_time(2 * TURN), pre);
                prefetch_aux_rows<EPI, MB, NB, 2 * TURN + 1>(g, aux_pos, at_run_time(2 * TURN + 1), pre);
            }
        float a[MB][8], b[NB][8];
#pragma unroll
        for (int mi = 0; mi < MB; ++mi) operand<A_KC, TM>(lds_a[cur], wm + 32 * mi + r32, half, a[mi]);
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) operand<B_KC, TN>(lds_b[cur], wn + 32 * ni + r32, half, b[ni]);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int mi = 0; mi < MB; ++mi)
#pragma unroll
                for (int ni = 0; ni < NB; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mi][kk], b[ni][kk], acc[mi][ni], 0, 0, 0);
        if (AHEAD > 1 || s + 1 < slabs) stash(cur ^ 1, ring_a[NEXT], ring_b[NEXT]);
        __syncthreads();
    };
    uint32_t s = 0;
    if constexpr (AHEAD > 1)
        for (; s + 8 <= slabs; s += 8) {
            iteration(s, Part<0>{}); iteration(s + 1, Part<1>{}); iteration(s + 2, Part<2>{}); iteration(s + 3, Part<3>{});
            iteration(s + 4, Part<4>{}); iteration(s + 5, Part<5>{}); iteration(s + 6, Part<6>{}); iteration(s + 7, Part<7>{});
        }
    for (; s < slabs; s += 8) {
        iteration(s, Part<0>{});
        if (s + 1 < slabs) iteration(s + 1, Part<1>{});
        if (s + 2 < slabs) iteration(s + 2, Part<2>{});
        if (s + 3 < slabs) iteration(s + 3, Part<3>{});
        if (s + 4 < slabs) iteration(s + 4, Part<4>{});
        if (s + 5 < slabs) iteration(s + 5, Part<5>{});
        if (s + 6 < slabs) iteration(s + 6, Part<6>{});
        if (s + 7 < slabs) iteration(s + 7, Part<7>{});
    }
    prefetch_aux_rest<EPI, MB, NB>(g, aux_pos, 2 * slabs, pre);    // K shorter than the parts

    epilogue<EPI, MB, NB>(g, t, acc, wm, wn, half, r32, full_tile, pre, lds_a[0]);
}

// weights -= lr x (sum over the batch of a^T b) for batches of up to 128 samples (BLOCKS x 32; 160 take
// as long either way): a streams the rows of the weight
// matrix, b its columns, both stored [sample][row or column].  A wave owns 32 columns of the matrix, whose operand stays in its
// registers, and goes down the rows in blocks of 32; the rows' operand passes through local memory for the four waves.
// Bound by the matrix cores.  As tiles with K = batch, eight slabs at batch 128, filling and draining each tile's pipeline lay
// open (matrix cores busy 67 % of the time against 89 % in the forward products); here nothing restarts between row blocks (79 %).
// 256 nodes, 1024 x 4096 weights, batch 128: 2.66 -> 2.45 ms, 2.07 for the matrix instructions alone.  Whole calls, two steps, us:
// that swarm, at the power limit, 24 380 -> 23 790 and 24 740 -> 24 420 in two runs; 32 nodes, 800-1504-480, batch 64 572 -> 537;
// 23 nodes, 448-3840-224, batch 96 1035 -> 954; 36 nodes, 608-1280-64, batch 128 537 -> 508; 48 nodes, 1024-4096-1024, batch 64
// 2901 -> 2817; 8 nodes at batch 32 the same.
// Three workgroups per compute unit: with four blocks of samples that costs 12 bytes of scratch per lane; two without it take
// as long (that swarm 2.42 and 2.46 ms for W1 and W2, 2.47 and 2.46 with two; 36 nodes, 608-1280-64: 84 and 14 us, 86 and 14).
// The order of the products is that of mlp_gemm_kernel, so is every bit.
// Below 128 samples the biases go along (BIASES): the workgroups of a block of rows take turns at its biases, whose gradient is the sum
// of the rows' operand over the samples (13 nodes, 704-416-64, batch 96, two steps: 147 -> 135 us with two launches fewer per step; by the first
// of the workgroups alone, with the bias read when it is due, an update of 256 x 4096 x 1024 took 2.91 ms instead of 2.55).  At 128
// samples it takes registers that are not there: 84.5 instead of 88 us at 8 nodes, 128-256-64, but 23 800 instead of 23 200 at 256
// nodes, 1024-4096-1024.
struct FloatUpdateArgs {
    const float *a, *b, *src;       // src: models, `d` floats per node
    float *dst;
    const uint32_t *nodes;
    uint64_t a_stride, b_stride, d, weights, biases;
    uint32_t lda, ldb, ldw, rows, cols;        // rows, cols: blocks of 32
    uint32_t parts, groups_n, groups;          // a workgroup takes four column blocks and a part of the rows
    float lr;
};
constexpr uint32_t STREAMED_SAMPLES = 128;
constexpr int ROW_LD = 36;                     // the two halves of a wave read different banks

template <int BLOCKS>
__global__ __launch_bounds__(256, 3) void mlp_float_update_kernel(const FloatUpdateArgs g) {
    constexpr int K = 32 * BLOCKS;
    constexpr bool BIASES = BLOCKS < 4;
    __shared__ __attribute__((aligned(16))) float lds[2][K * ROW_LD];
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, r32 = lane & 31u, wave = wave_of_group();
    bool valid;
    const uint32_t q = place_of(blockIdx.x, g.groups, valid);
    if (!valid) return;
    const uint32_t per_slot = g.groups_n * g.parts, slot = q / per_slot, part = q % per_slot / g.groups_n, group = q % g.groups_n;
    const uint32_t node = g.nodes ? g.nodes[slot] : slot, ldw = g.ldw;
    const bool live = group * 4 + wave < g.cols;
    const uint32_t col = live ? group * 4 + wave : g.cols - 1;
    const uint32_t first = (uint32_t)((uint64_t)g.rows * part / g.parts), last = (uint32_t)((uint64_t)g.rows * (part + 1) / g.parts);
    const float *a = g.a + slot * g.a_stride, *b = g.b + slot * g.b_stride + 32 * col;
    const float *src = g.src + node * g.d + g.weights + 32 * col;
    float *dst = g.dst + node * g.d + g.weights + 32 * col;
    const uint32_t lane_bytes = 4 * (4 * half * ldw + r32), row = threadIdx.x >> 3, at = 4 * (threadIdx.x & 7u);

    auto at_bias = [&](uint32_t r) {
        uint32_t t = threadIdx.x;
        asm volatile("" : "+v"(t));              // made where it is used: registers are short
        return node * g.d + g.biases + 32 * r + (t >> 3);
    };
    auto load_rows = [&](uint32_t r, f4 v[BLOCKS]) {                 // thread t: 4 rows of sample t / 8 of every 32
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) v[i] = *(const f4 *)(a + (uint64_t)(32 * i + row) * g.lda + 32 * r + at);
    };
    auto keep_rows = [&](float *to, const f4 v[BLOCKS]) {
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) *(f4 *)(to + (32 * i + row) * ROW_LD + at) = v[i];
    };
    auto load_weights = [&](uint32_t r, float w[16]) {
        const Buffer from = buffer_at(src + (uint64_t)32 * r * ldw, 128 * (uint64_t)ldw);
#pragma unroll
        for (int v = 0; v < 16; ++v) w[v] = load4(from, lane_bytes, 4 * row_of(v, 0) * ldw);
    };

    float columns[K / 2];                      // samples 16 f + 8 half + j of column r32 at 8 f + j
    constexpr int AD = BLOCKS <= 3 ? 2 : 1;    // row blocks of operands on their way, as the registers allow
    f4 staged[AD][BLOCKS];
    float w[2][16];
    load_rows(first, staged[0]);
    if (AD == 2) load_rows(min(first + 1, last - 1), staged[AD - 1]);
#pragma unroll
    for (int f = 0; f < K / 16; ++f)
#pragma unroll
        for (int j = 0; j < 8; ++j) columns[8 * f + j] = b[(uint64_t)(16 * f + 8 * half + j) * g.ldb + r32];
    load_weights(first, w[0]);
    keep_rows(lds[0], staged[0]);
    __syncthreads();
    uint32_t next_biases = first + (group + g.groups_n - first % g.groups_n) % g.groups_n;       // row block r is group r % groups_n's
    // Row block r.  Loads and stores complete in order: what is waited for at the end of a block is better not requested after
    // the block before was stored, hence the second block of operands on its way.
    auto step = [&](uint32_t r, auto parity) {
        constexpr int PARITY = decltype(parity)::value;
        float (&now)[16] = w[PARITY], (&ahead)[16] = w[!PARITY];
        const float *rows = lds[PARITY] + 8 * half * ROW_LD + r32;
        load_rows(min(r + AD, last - 1), staged[PARITY % AD]);
        load_weights(min(r + 1, last - 1), ahead);
        // the rows' biases, a block's by one workgroup in turn: thread t a share of row t / 8, every eighth sample
        const bool biased = BIASES && r == next_biases;
        if (biased) next_biases += g.groups_n;
        float share = 0.f, bias = 0.f;
        if (biased) {
            bias = g.src[at_bias(r)];
#pragma unroll
            for (int i = 0; i < K / 8; ++i) share += lds[PARITY][(8 * i + (lane & 7u)) * ROW_LD + row];
            share += across<1>(share);
            share += across<2>(share);
            share += across<4>(share);
        }
        __builtin_amdgcn_sched_barrier(0);
        f16v sum = cleared();
#pragma unroll
        for (int f = 0; f < K / 16; ++f)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                sum = __builtin_amdgcn_mfma_f32_32x32x2f32(rows[(16 * f + j) * ROW_LD], columns[8 * f + j], sum, 0, 0, 0);
        if (live) {
            const Buffer to = buffer_at(dst + (uint64_t)32 * r * ldw, 128 * (uint64_t)ldw);
#pragma unroll
            for (int v = 0; v < 16; ++v) store4(to, fmaf(-g.lr, sum[v], now[v]), lane_bytes, 4 * row_of(v, 0) * ldw);
        }
        if (biased && (lane & 7u) == 0) g.dst[at_bias(r)] = fmaf(-g.lr, share, bias);
        keep_rows(lds[!PARITY], staged[(PARITY + 1) % AD]);
        __syncthreads();
    };
    uint32_t r = first;
    for (; r + 1 < last; r += 2) {
        step(r, std::integral_constant<int, 0>{});
        step(r + 1, std::integral_constant<int, 1>{});
    }
    if (r < last) step(r, std::integral_constant<int, 0>{});
}

static void launch_float_update(FloatUpdateArgs g, uint32_t batch, uint32_t count, hipStream_t st) {
    g.groups_n = parts_of(g.cols, 4);
    // up to 1024 workgroups a block of rows each, else two or more (us for two steps of one node, two or more throughout and so:
    // 608-1280-64, batch 128 234 and 227; 800-1504-480, batch 64 210 and 203; 39 nodes, 96-256-64, batch 128 124 and 120)
    g.parts = (uint64_t)count * g.groups_n * g.rows <= 1024 ? g.rows : std::max(1u, std::min(1024 / (count * g.groups_n), g.rows / 2));
    g.groups = g.groups_n * g.parts * count;
    const uint32_t grid = whole_turns(g.groups);
    switch (batch / 32) {
        case 1: mlp_float_update_kernel<1><<<grid, 256, 0, st>>>(g); break;
        case 2: mlp_float_update_kernel<2><<<grid, 256, 0, st>>>(g); break;
        case 3: mlp_float_update_kernel<3><<<grid, 256, 0, st>>>(g); break;
        default: mlp_float_update_kernel<4><<<grid, 256, 0, st>>>(g); break;
    }
}

// A minibatch (mlp_batch.hpp).  Every thread searches the label of its own sample (the threads of a sample read the same
// ten or so words one after the other), which costs less than a launch of its own for the labels: 5 us per step.
__global__ __launch_bounds__(256) void mlp_batch_kernel(const float *__restrict__ means, const float *__restrict__ cdf,
                                                        const uint32_t *__restrict__ nodes, const uint32_t *__restrict__ events,
                                                        uint32_t *__restrict__ labels, float *__restrict__ x, uint32_t n_in,
                                                        uint32_t n_out, uint32_t batch, float sigma, uint64_t seed,
                                                        uint32_t event, uint32_t q) {
    const uint32_t slot = blockIdx.y, node = nodes ? nodes[slot] : slot;
    if (events) event = events[slot];
    const uint64_t f = (uint64_t)blockIdx.x * 256 + threadIdx.x;       // float4 index within the batch
    if (f * 4 >= (uint64_t)batch * n_in) return;
    const uint32_t s = (uint32_t)(f * 4 / n_in), k = (uint32_t)(f * 4 % n_in);
    const uint32_t y = sample_label(cdf + (uint64_t)node * n_out, n_out, seed, q, node, event, s);
    if (k == 0) labels[(uint64_t)slot * batch + s] = y;
    *(f4 *)(x + ((uint64_t)slot * batch + s) * n_in + k) = sample_features(means + (uint64_t)y * n_in + k, sigma, seed, q, node, event, f);
}

__device__ __forceinline__ float block_reduce(float v, float *lds, bool is_max) {
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(v, off);
        v = is_max ? fmaxf(v, o) : v + o;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = lds[0];
    for (uint32_t w = 1; w < blockDim.x / 64; ++w) r = is_max ? fmaxf(r, lds[w]) : r + lds[w];
    return r;
}

// In place: logits row -> (softmax - onehot(y)) / batch.  Rows of up to 2048 entries stay in registers between
// the three passes (maximum, sum of exponentials, result): one read and one write of the row.
// Logits in parts (up to 2048 classes): their sum and the bias come first.
struct LogitParts {
    const float *first, *bias;       // first: part 0 of slot 0; bias: of node 0
    const uint32_t *nodes;
    uint64_t slot_stride, part_stride, d;
    uint32_t parts;
};
constexpr uint32_t PARTED_CLASSES = 2048;

template <bool PARTED>
__global__ __launch_bounds__(256) void mlp_softmax_grad_kernel(float *__restrict__ logits,
                                                               const uint32_t *__restrict__ labels, uint32_t n_out,
                                                               uint32_t batch, const LogitParts lp) {
    __shared__ float lds[4];
    const uint32_t slot = blockIdx.y, s = blockIdx.x;
    float *row = logits + ((uint64_t)slot * batch + s) * n_out;
    const uint32_t y = labels[(uint64_t)slot * batch + s];
    const float inv_b = 1.0f / (float)batch;
    auto whole = [&](uint32_t c) {
        const float *p = lp.first + slot * lp.slot_stride + (uint64_t)s * n_out + c;
        float sum = p[0];
        for (uint32_t i = 1; i < lp.parts; ++i) sum += p[i * lp.part_stride];
        return sum + lp.bias[(lp.nodes ? lp.nodes[slot] : slot) * lp.d + c];
    };
    constexpr int HELD = PARTED_CLASSES / 256;
    if (PARTED || n_out <= 256 * HELD) {
        float v[HELD];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            const uint32_t c = threadIdx.x + 256 * i;
            v[i] = c < n_out ? (PARTED ? whole(c) : row[c]) : -INFINITY;
            mx = fmaxf(mx, v[i]);
        }
        mx = block_reduce(mx, lds, true);
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            v[i] = expf(v[i] - mx);              // exp(-inf) = 0 for the entries past the row
            sum += v[i];
        }
        sum = block_reduce(sum, lds, false);
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            const uint32_t c = threadIdx.x + 256 * i;
            if (c < n_out) row[c] = (v[i] / sum - (c == y ? 1.f : 0.f)) * inv_b;
        }
        return;
    }
    float mx = -INFINITY;
    for (uint32_t c = threadIdx.x; c < n_out; c += 256) mx = fmaxf(mx, row[c]);
    mx = block_reduce(mx, lds, true);
    float sum = 0.f;
    for (uint32_t c = threadIdx.x; c < n_out; c += 256) sum += expf(row[c] - mx);
    sum = block_reduce(sum, lds, false);
    for (uint32_t c = threadIdx.x; c < n_out; c += 256)
        row[c] = (expf(row[c] - mx) / sum - (c == y ? 1.f : 0.f)) * inv_b;
}

// b_dst = b_src - lr * column sums of G (batch x width): 64 columns per workgroup, each wave takes every fourth row
// (batch is a multiple of 32), eight loads in flight.
__global__ __launch_bounds__(256) void mlp_bias_kernel(const float *__restrict__ G, const float *__restrict__ src,
                                                       float *__restrict__ dst, const uint32_t *__restrict__ nodes,
                                                       uint32_t width, uint32_t batch, uint64_t d, uint64_t bias_off,
                                                       float lr) {
    __shared__ float part[4][64];
    const uint32_t slot = blockIdx.y, node = nodes ? nodes[slot] : slot;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, c = blockIdx.x * 64 + lane;
    const float *g = G + (uint64_t)slot * batch * width + min(c, width - 1);
    float sum = 0.f;
    for (uint32_t s = wave; s < batch; s += 32) {
        float v[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) v[i] = g[(uint64_t)(s + 4 * i) * width];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) sum += v[i];
    }
    part[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || c >= width) return;
    sum = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    dst[(uint64_t)node * d + bias_off + c] = fmaf(-lr, sum, src[(uint64_t)node * d + bias_off + c]);
}

static void launch_mlp_bias(const float *G, const float *src, float *dst, const uint32_t *nodes, uint32_t width, uint32_t batch,
                            uint32_t count, uint64_t d, uint64_t bias_off, float lr, hipStream_t st) {
    mlp_bias_kernel<<<dim3((width + 63) / 64, count), 256, 0, st>>>(G, src, dst, nodes, width, batch, d, bias_off, lr);
}

hipError_t alloc_mlp(MlpObjective &o, uint32_t n_nodes) {
    o.n_nodes = n_nodes;
    const size_t b = o.batch;
    hipError_t e;
    if ((e = hipMalloc((void **)&o.x, sizeof(float) * n_nodes * b * o.n_in)) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&o.hid, sizeof(float) * n_nodes * b * o.n_hid)) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&o.dlogits, sizeof(float) * n_nodes * b * o.n_out)) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&o.dhid, sizeof(float) * n_nodes * b * o.n_hid)) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&o.labels, sizeof(uint32_t) * n_nodes * b)) != hipSuccess) return e;
    return hipSuccess;
}

void free_mlp(MlpObjective &o) {
    void *p[] = {o.x, o.hid, o.dlogits, o.dhid, o.labels};
    for (void *q : p) if (q) (void)hipFree(q);
    free_mlp_split(o);
    o = MlpObjective{};
}

template <bool A_KC, bool B_KC, int EPI, int TM, int TN>
static void gemm_tiled(GemmArgs g, uint32_t count, hipStream_t st) {
    g.tiles_n = (g.N + TN - 1) / TN;
    g.tiles_m = (g.M + TM - 1) / TM;
    g.groups = g.tiles_n * g.tiles_m * count * (EPI == EPI_PART ? g.parts : 1u);
    const dim3 grid(8 * ((g.groups + 7) / 8), 1, 1);          // a whole number of turns over the dies
    mlp_gemm_kernel<A_KC, B_KC, EPI, TM, TN><<<grid, tile_threads(TM), 0, st>>>(g);
}

// Tile of a product, by its shape and, where that decides whether the tiles fill the chip, the number of nodes in the launch
// (the order of every sum is the same in all of them).  Tiles of 128 x 128 read the fewest operand bytes and issue the fewest
// instructions per product; smaller ones where they would be mostly padding or too few to fill the chip (two fit a
// compute unit).  M is the batch in the forward and backward products:
//  - 32 and 96 rows: 32 x 64 by two waves, without padding (us for two steps, tiles of 64 and 128 rows and so: batch 96, 50 nodes,
//    800-1504-480 1225 -> 1097, 13 nodes, 704-416-64 163 -> 147; batch 32, 49 nodes, 224-1440-64 200 -> 184; a tile of 96 rows: 1163, 182),
//    at 96 rows where tiles of 128 x 128 do not fill their turns (below).  At 160 rows the weights' third and further reads cost more than the padding (20 nodes, 320-512-800: 338 and 372);
//  - 64 rows: 64 x 64.  32 nodes, 800-1504-480, batch 64, two steps (with the other small kernels of this file):
//    937 -> 635 us; 8 nodes, 1024-4096-1024, batch 32: 1115 -> 679;
//  - 129 to 192 rows and the like: three tiles of 64 rows instead of two of 128 (64 nodes, 736-1376-896, batch 160:
//    3259 -> 2770 us).  The same remainder above 192 rows, all rules together against 128 x 128 throughout: 32 nodes,
//    800-1504-480, batch 288 2380 -> 1837, 320 2492 -> 1907; 16 nodes, 1024-4096-1024, batch 544 7350 -> 6544; 8 nodes,
//    batch 1056 7417 -> 6231;
//  - fewer than 512 tiles of 128 x 128: 128 x 64 (4 nodes, 1024-2048-512, batch 128: 648 -> 433 us); so where more of them leave over a
//    fifth of their turns of 512 empty (50 nodes, 800-1504-480, batch 128, 600 tiles in two turns: 1323 -> 1270; 60 nodes,
//    704-1632-512, 780: 1600 -> 1545.  Full turns: 64 nodes, 512-4096-1024, batch 96, logits in 512 tiles 579 us, 648 by tiles of 32 rows).
// The update products of batches above 128 take 64 x 64 below 256 tiles; above, the smaller tile's extra operand reads cost
// more than it brings.
static int tile_rows(uint32_t batch) {
    if (batch == 32 || batch == 96) return 32;
    const uint32_t over = batch % 128;
    return batch <= 64 || (over != 0 && over <= 64) ? 64 : 128;
}

template <bool A_KC, bool B_KC, int EPI>
static void gemm(const GemmArgs &g, uint32_t count, hipStream_t st) {
    const uint32_t large = ((g.M + 127) / 128) * ((g.N + 127) / 128) * count;
    if constexpr (EPI == EPI_SGD_UPDATE) {
        if (large < 256) gemm_tiled<A_KC, B_KC, EPI, 64, 64>(g, count, st);
        else gemm_tiled<A_KC, B_KC, EPI, 128, 128>(g, count, st);
    } else {
        const bool fill = large >= 512 && 5 * large >= 4 * 512 * parts_of(large, 512);
        if (tile_rows(g.M) == 32 && (g.M == 32 || !fill)) gemm_tiled<A_KC, B_KC, EPI, 32, 64>(g, count, st);
        else if (tile_rows(g.M) == 64) gemm_tiled<A_KC, B_KC, EPI, 64, 64>(g, count, st);
        else if (EPI == EPI_PART || !fill) gemm_tiled<A_KC, B_KC, EPI, 128, 64>(g, count, st);
        else if constexpr (EPI != EPI_PART) gemm_tiled<A_KC, B_KC, EPI, 128, 128>(g, count, st);
    }
}

// Parts that the logits' product is cut into along the hidden units, by the swarm and not by the nodes of a launch (a node's bits
// do not depend on who steps along): as many as make 512 workgroups of 64 rows and 64 classes, each of 64 units or more, as far as
// the gradient of the hidden units, which is made later, has room for them.  us for two steps, whole and in parts (with the other
// changes of small steps in this file): 12 nodes, 512-2048-64, batch 32 261 -> 142, of which the product 67 -> 7 and the softmax
// 5 -> 11; 7 nodes, 96-3072-544, batch 128 504 -> 317; 30 nodes, 256-704-192, batch 64 180 -> 151.
static uint32_t logit_parts(const MlpObjective &o, uint32_t n) {
    if (o.n_out > PARTED_CLASSES) return 1;
    const uint64_t tiles = (uint64_t)n * parts_of(o.batch, 64) * parts_of(o.n_out, 64);
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({512 / tiles, o.n_hid / 64, o.n_hid / o.n_out}));
}

hipError_t launch_local_mlp(const float *base, float *W, const MlpObjective &o, const LocalSlots &slots,
                            uint32_t count, uint32_t n, uint64_t d, uint32_t H, float lr, uint64_t seed,
                            uint32_t event, hipStream_t st) {
    const uint32_t *nodes = slots.nodes;          // the number of steps is constant for this objective
    if (count == 0) return hipSuccess;
    if (o.bf16x3) return launch_local_mlp_split(base, W, o, slots, count, d, H, lr, seed, event, st);
    const uint32_t I = o.n_in, Hd = o.n_hid, O = o.n_out, Bt = o.batch;
    const uint64_t off_b1 = (uint64_t)Hd * I, off_w2 = off_b1 + Hd, off_b2 = off_w2 + (uint64_t)O * Hd;
    const uint32_t parts = logit_parts(o, n);
    const bool biases_inside = Bt < STREAMED_SAMPLES;      // with the updates
    for (uint32_t q = 0; q < H; ++q) {
        const float *src = q == 0 ? base : W;
        mlp_batch_kernel<<<dim3((unsigned)(((uint64_t)Bt * I / 4 + 255) / 256), count), 256, 0, st>>>(
            o.means, o.cdf, nodes, slots.events, o.labels, o.x, I, O, Bt, o.data_sigma, seed, event, q);
        GemmArgs g{};
        g.nodes = nodes; g.lr = lr;
        // hid = relu(x W1^T + b1):  M = batch, N = hid, K = in
        g.A = o.x; g.strideA = (uint64_t)Bt * I; g.a_by_node = 0; g.lda = I;
        g.B = src; g.strideB = d; g.b_by_node = 1; g.ldb = I;
        g.C = o.hid; g.strideC = (uint64_t)Bt * Hd; g.c_by_node = 0; g.ldc = Hd;
        g.aux = src + off_b1; g.strideAux = d; g.aux_by_node = 1; g.ldaux = 0;
        g.M = Bt; g.N = Hd; g.K = I;
        gemm<true, true, EPI_BIAS_RELU>(g, count, st);
        // logits = hid W2^T + b2:  M = batch, N = out, K = hid
        g.A = o.hid; g.strideA = (uint64_t)Bt * Hd; g.lda = Hd;
        g.B = src + off_w2; g.ldb = Hd;
        g.C = o.dlogits; g.strideC = (uint64_t)Bt * O; g.ldc = O;
        g.aux = src + off_b2;
        g.M = Bt; g.N = O; g.K = Hd;
        LogitParts lp{o.dhid, src + off_b2, nodes, (uint64_t)Bt * Hd, (uint64_t)Bt * O, d, 1};
        const dim3 rows(Bt, count);
        if (parts > 1) {
            g.C = o.dhid; g.strideC = lp.slot_stride;
            g.part_k = parts_of(Hd / TK, parts) * TK; g.parts = lp.parts = parts_of(Hd, g.part_k); g.part_stride = lp.part_stride;
            gemm<true, true, EPI_PART>(g, count, st);
            mlp_softmax_grad_kernel<true><<<rows, 256, 0, st>>>(o.dlogits, o.labels, O, Bt, lp);
        } else {
            gemm<true, true, EPI_BIAS>(g, count, st);
            mlp_softmax_grad_kernel<false><<<rows, 256, 0, st>>>(o.dlogits, o.labels, O, Bt, lp);
        }
        // dpre = (dlogits W2) * [hid > 0]:  M = batch, N = hid, K = out;  W2 stored [k][n]
        g.A = o.dlogits; g.strideA = (uint64_t)Bt * O; g.lda = O;
        g.B = src + off_w2; g.ldb = Hd;
        g.C = o.dhid; g.strideC = (uint64_t)Bt * Hd; g.ldc = Hd;
        g.aux = o.hid; g.strideAux = (uint64_t)Bt * Hd; g.aux_by_node = 0; g.ldaux = Hd;
        g.M = Bt; g.N = Hd; g.K = O;
        if (Bt == STREAMED_SAMPLES) { g.colsum_src = src + off_b1; g.colsum_dst = W + off_b1; g.strideColsum = d; }
        gemm<true, false, EPI_RELU_MASK>(g, count, st);
        g.colsum_src = nullptr; g.colsum_dst = nullptr;
        // W2 <- W2 - eta dlogits^T hid,  W1 <- W1 - eta dpre^T x;  all operands stored [sample][row]
        if (Bt <= STREAMED_SAMPLES) {
            FloatUpdateArgs u{};
            u.nodes = nodes; u.src = src; u.dst = W; u.d = d; u.lr = lr;
            u.a = o.dlogits; u.a_stride = (uint64_t)Bt * O; u.lda = O;
            u.b = o.hid; u.b_stride = (uint64_t)Bt * Hd; u.ldb = Hd;
            u.weights = off_w2; u.biases = off_b2; u.ldw = Hd; u.rows = O / 32; u.cols = Hd / 32;
            launch_float_update(u, Bt, count, st);
            u.a = o.dhid; u.a_stride = (uint64_t)Bt * Hd; u.lda = Hd;
            u.b = o.x; u.b_stride = (uint64_t)Bt * I; u.ldb = I;
            u.weights = 0; u.biases = off_b1; u.ldw = I; u.rows = Hd / 32; u.cols = I / 32;
            launch_float_update(u, Bt, count, st);
        } else {
            g.A = o.dlogits; g.strideA = (uint64_t)Bt * O; g.a_by_node = 0; g.lda = O;
            g.B = o.hid; g.strideB = (uint64_t)Bt * Hd; g.b_by_node = 0; g.ldb = Hd;
            g.C = W + off_w2; g.strideC = d; g.c_by_node = 1; g.ldc = Hd;
            g.aux = src + off_w2; g.strideAux = d; g.aux_by_node = 1; g.ldaux = Hd;
            g.M = O; g.N = Hd; g.K = Bt;
            gemm<false, false, EPI_SGD_UPDATE>(g, count, st);
            g.A = o.dhid; g.strideA = (uint64_t)Bt * Hd; g.lda = Hd;
            g.B = o.x; g.strideB = (uint64_t)Bt * I; g.ldb = I;
            g.C = W; g.ldc = I;
            g.aux = src; g.ldaux = I;
            g.M = Hd; g.N = I; g.K = Bt;
            gemm<false, false, EPI_SGD_UPDATE>(g, count, st);
        }
        if (!biases_inside) launch_mlp_bias(o.dlogits, src, W, nodes, O, Bt, count, d, off_b2, lr, st);
        if (Bt > STREAMED_SAMPLES) launch_mlp_bias(o.dhid, src, W, nodes, Hd, Bt, count, d, off_b1, lr, st);
    }
    return hipGetLastError();
}

}  // namespace swarm
