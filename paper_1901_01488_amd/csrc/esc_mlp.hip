// esc_mlp.hip -- the learned cardinality estimator of the gate: an MLP
// 64 -> 256 -> 256 -> 256 -> 1 (ReLU) trained and run on the GPU with
// bfloat16 MFMA operands (v_mfma_f32_32x32x16_bf16) and float32 accumulation.
//
// The paper replaces estimates from synopses by exact counts (Section 2);
// the estimator here only decides which predicates need that exact count,
// and exact counts computed by the scan are its training labels.
//
// Rounding points (identical in the CPU oracle): every GEMM operand is
// bfloat16 (round to nearest even): the features, the weights, the hidden
// activations handed to the next layer and the back-propagated deltas;
// bias adds, ReLU, the head and all reductions are float32.  The ReLU
// derivative is taken from the rounded activation (> 0).
//
// Memory (all caller-owned): the state holds the float32 master weights,
// the Adam moments, the step counters and bfloat16 copies of the weights
// packed in MFMA B-operand fragment order (each wave's fragment of a
// 32-column tile and a 16-deep k step is one contiguous 1 KiB block, read
// with one 16-byte load per lane); for the backward products W2 and W3 are
// also packed transposed.  The training workspace holds the transposed
// activations and deltas of one batch and per-block partial sums.
//
// Kernels (a block is 8 waves; wave w owns output columns 32w .. 32w+31 of
// every 256-wide layer):
//   forward_kernel<MT>: 32*MT rows per block; all four layers in one launch,
//     activations in LDS between layers, weights straight from L2;
//   train_rows_kernel: 32 rows per block; gathers the minibatch, runs the
//     forward, the head with the Huber-loss derivative and the two backward
//     products, keeps every activation and delta in LDS, stores them
//     transposed (feature-major) for the weight gradients, and writes
//     per-block column sums (bias gradients), head-gradient and loss
//     partials;
//   weight_grad_kernel<ADAM>: one 32x32 tile of a weight gradient per block
//     (a product over the batch rows), with Adam applied in the epilogue
//     (master weights, moments and both bf16 packings refreshed); five extra
//     blocks sum the partials over blocks in a fixed order for the biases,
//     W4, b4 and the loss.
// A training step is these two launches.  Every reduction has a fixed order,
// so training is deterministic run to run.  At batch 256 a step is bound by
// the latency of its dependent loads and layer steps and by each of the 8 rows
// blocks reading 560 KB of weights through one CU's L1.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "esc_host.h"
#include "esc_runtime.h"

namespace esc {

constexpr int kIn = 64, kHid = 256;
constexpr int kMaxBatch = 4096;
constexpr float kHuber = 0.5f;   // Huber loss threshold on ln(selectivity) errors

// flat parameter layout (float32): W1, b1, W2, b2, W3, b3, W4, b4
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kIn * kHid;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid * kHid;
constexpr int kOffW4 = kOffB3 + kHid;
constexpr int kOffB4 = kOffW4 + kHid;
constexpr int kNParams = kOffB4 + 1;
static_assert(kNParams == ESC_MLP_NPARAMS, "parameter count");

// bf16 packings (element offsets): forward W1..W3, transposed W2 and W3, W4
constexpr int kPkF1 = 0;
constexpr int kPkF2 = kPkF1 + kIn * kHid;
constexpr int kPkF3 = kPkF2 + kHid * kHid;
constexpr int kPkB2 = kPkF3 + kHid * kHid;
constexpr int kPkB3 = kPkB2 + kHid * kHid;
constexpr int kPkW4 = kPkB3 + kHid * kHid;
constexpr int kNPack = kPkW4 + kHid;

constexpr size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// state layout (bytes)
constexpr size_t kStP = 0;
constexpr size_t kStM = up256(kStP + (size_t)kNParams * 4);
constexpr size_t kStV = up256(kStM + (size_t)kNParams * 4);
constexpr size_t kStSteps = up256(kStV + (size_t)kNParams * 4);   // int64 [0] Adam steps, [1] unused
constexpr size_t kStHyper = kStSteps + 64;                          // lr, b1, b2, eps
constexpr size_t kStPack = up256(kStHyper + 64);
constexpr size_t kStateBytes = up256(kStPack + (size_t)kNPack * 2);

// per-block partial sums of the training rows kernel (floats)
constexpr int kPartColsum = 0;               // [3][256] column sums of the layer deltas (bias gradients)
constexpr int kPartW4 = 3 * kHid;            // [256] head weight gradient
constexpr int kPartB4 = kPartW4 + kHid;      // head bias gradient
constexpr int kPartLoss = kPartB4 + 1;       // sum of the rows' losses
constexpr int kPartStride = kPartLoss + 7;   // 1032 floats per block

typedef uint16_t bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__host__ __device__ __forceinline__ float bf2f(bf16_t h)
{
    uint32_t u = (uint32_t)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

// round to nearest even (v_cvt_pk_bf16_f32: the same as adding half of the last
// place in integers, on every one of the 2^32 bit patterns, in one op for eight)
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

// Element offset of B(k, n) of a K x N matrix in fragment order: fragment
// (n/32, k/16) is 64 lanes x 8 values, lane = 32 (k/8 % 2) + n % 32, value
// k % 8 (the B operand of v_mfma_f32_32x32x16_bf16).
__host__ __device__ __forceinline__ int frag_off(int k, int n, int K)
{
    return ((((n >> 5) * (K >> 4) + (k >> 4)) * 64 + ((k >> 3) & 1) * 32 + (n & 31)) << 3) + (k & 7);
}

struct Hyper {
    float lr, b1, b2, eps;
};

struct State {
    float *p, *m, *v;
    long long *steps;
    Hyper *hyper;
    bf16_t *pk;
};

struct TrainWs {
    bf16_t *aT[3];   // layer inputs, transposed: [fan_in][bp]
    bf16_t *gT[3];   // rounded deltas of layers 1..3, transposed: [256][bp]
    float *part;     // [blocks][kPartStride]
};

constexpr int kBlock = 512;   // 8 waves
constexpr int kWaves = kBlock / 64;
constexpr int LDA = kHid + 8;   // LDS row stride (bf16) of 256-wide activations: +16 bytes
constexpr int LDX = kIn + 8;

size_t train_ws_bytes(int batch, TrainWs *ws, char *base)
{
    const size_t bp = (size_t)((batch + 31) / 32 * 32);
    const size_t nb = bp / 32;
    size_t off = 0;
    const size_t sizes[6] = {kIn * bp * 2, kHid * bp * 2, kHid * bp * 2, kHid * bp * 2, kHid * bp * 2, kHid * bp * 2};
    char *ptr[6];
    for (int i = 0; i < 6; i++) {
        ptr[i] = base ? base + off : nullptr;
        off = up256(off + sizes[i]);
    }
    if (ws) {
        for (int i = 0; i < 3; i++) ws->aT[i] = (bf16_t *)ptr[i];
        for (int i = 0; i < 3; i++) ws->gT[i] = (bf16_t *)ptr[3 + i];
        ws->part = base ? (float *)(base + off) : nullptr;
    }
    off = up256(off + nb * kPartStride * 4);
    return off;
}

// ------------------------------------------------------------------ device helpers

__device__ __forceinline__ int lane_of() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_of() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// A barrier for data in LDS alone: global loads and stores stay in flight over
// it (__syncthreads waits for all of them, and so for the next layers' weights).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A wave's B fragments of one layer (K deep, columns 32 nt ..), packed in
// fragment order in global memory: KS 16-byte loads per lane, all in flight.
template <int K>
__device__ __forceinline__ void load_frags(const bf16_t *Bpk, int nt, u16x8 (&b)[K / 16])
{
    constexpr int KS = K / 16;
    const u16x8 *src = (const u16x8 *)Bpk + (size_t)nt * KS * 64 + lane_of();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) b[ks] = src[ks * 64];
}

// acc[mt] = A(rows 32 mt .. 32 mt + 31, 0..K) * B(0..K, the wave's columns),
// A in LDS (bf16, row stride lda).
template <int MT, int K>
__device__ __forceinline__ void mma_layer(const bf16_t *As, int lda, const u16x8 (&b)[K / 16], f32x16 (&acc)[MT])
{
    constexpr int KS = K / 16;
    const int lane = lane_of();
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc[mt][i] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const u16x8 a = *(const u16x8 *)&As[(32 * mt + (lane & 31)) * lda + 16 * ks + 8 * (lane >> 5)];
            acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                              __builtin_bit_cast(bf16x8, b[ks]), acc[mt], 0, 0, 0);
        }
    }
}

// accumulator element e of a lane: row 8 (e/4) + 4 (lane/32) + e%4, column lane%32
__device__ __forceinline__ int acc_row(int e) { return 8 * (e >> 2) + 4 * (lane_of() >> 5) + (e & 3); }

// four rows m .. m + 3 of feature n, bf16, as one 8-byte store into T[n][col0 + m]
__device__ __forceinline__ void store4(bf16_t *T, size_t ldt, int n, int col, const uint16_t (&v)[4])
{
    *(uint2 *)&T[(size_t)n * ldt + col] =
        make_uint2((uint32_t)v[0] | (uint32_t)v[1] << 16, (uint32_t)v[2] | (uint32_t)v[3] << 16);
}

// H[m][n] = bf16(relu(acc + bn)) for the wave's column tile (bn: the lane's
// column's bias); with T, also
// T[n][col0 + m] (an accumulator's elements are four consecutive rows of a
// feature, so the transposed copy needs no pass over LDS)
template <int MT>
__device__ __forceinline__ void store_relu(const f32x16 (&acc)[MT], int nt, float bn, bf16_t *Hs,
                                           bf16_t *T = nullptr, size_t ldt = 0, int col0 = 0)
{
    const int n = 32 * nt + (lane_of() & 31);
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            uint16_t h[4];
            const int m0 = 32 * mt + acc_row(4 * q);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float z = acc[mt][4 * q + e] + bn;
                h[e] = f2bf(z > 0.0f ? z : 0.0f);
                Hs[(m0 + e) * LDA + n] = h[e];
            }
            if (T) store4(T, ldt, n, col0 + m0, h);
        }
}

// dz = acc masked by (activation > 0); G[m][n] = bf16(dz) (Gs, if not null) and
// T[n][col0 + m] likewise; colsum[n] = sum of dz over the 32 rows (fixed order)
__device__ __forceinline__ void store_masked(const f32x16 &acc, int nt, const bf16_t *Mask, bf16_t *Gs, bf16_t *T,
                                             size_t ldt, int col0, float *colsum)
{
    const int lane = lane_of();
    const int n = 32 * nt + (lane & 31);
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        uint16_t g[4];
        const int m0 = acc_row(4 * q);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float dz = bf2f(Mask[(m0 + e) * LDA + n]) > 0.0f ? acc[4 * q + e] : 0.0f;
            s += dz;
            g[e] = f2bf(dz);
            if (Gs) Gs[(m0 + e) * LDA + n] = g[e];
        }
        store4(T, ldt, n, col0 + m0, g);
    }
    s += __shfl_xor(s, 32, 64);
    if (lane < 32) colsum[n] = s;
}

// y of rows m0, m0 + step, ..: a3[m] . bf16(W4) + b4 (whole wave; results in
// every lane), w4 holding the lane's four weights; the rows' reductions run
// side by side
template <int N>
__device__ __forceinline__ void head_rows(const bf16_t *A3, int m0, int step, const bf16_t (&w4)[4], float b4, float (&y)[N])
{
    const int lane = lane_of();
#pragma unroll
    for (int i = 0; i < N; i++) {
        y[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; j++) y[i] += bf2f(A3[(m0 + i * step) * LDA + lane + 64 * j]) * bf2f(w4[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int i = 0; i < N; i++) y[i] += __shfl_xor(y[i], o, 64);
#pragma unroll
    for (int i = 0; i < N; i++) y[i] += b4;
}

// T[f][col0 + r] = S[r][f] for r < 32, f < nf: each thread moves 8 rows of
// one feature as one 16-byte store
__device__ __forceinline__ void store_transposed(const bf16_t *S, int lds, int nf, bf16_t *T, size_t ldt, int col0)
{
    for (int it = threadIdx.x; it < nf * 4; it += kBlock) {
        const int f = it >> 2, r0 = (it & 3) * 8;
        u16x8 v;
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = S[(r0 + j) * lds + f];
        *(u16x8 *)&T[(size_t)f * ldt + col0 + r0] = v;
    }
}

// ------------------------------------------------------------------ inference

// yhat for rows [32 MT blockIdx.x, +32 MT) of X (n x 64 float32).  A layer's
// weights are loaded as it begins (all of them at the start, in 174 registers
// against 61: 6.8 against 6.2 us for 4,096 rows, 199 against 115 us for 262,144).
template <int MT>
__global__ __launch_bounds__(kBlock) void forward_kernel(const float *__restrict__ X, int64_t n,
                                                         const float *__restrict__ p, const bf16_t *__restrict__ pk,
                                                         float *__restrict__ yhat)
{
    constexpr int R = 32 * MT;
    __shared__ __attribute__((aligned(16))) bf16_t xs[R * LDX];
    __shared__ __attribute__((aligned(16))) bf16_t h0[R * LDA];
    __shared__ __attribute__((aligned(16))) bf16_t h1[R * LDA];
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int w = wave_of();
    // the input rows first: they are needed first
    constexpr int PER = R * kIn / kBlock;
    float x[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const int i = threadIdx.x + q * kBlock, m = i >> 6, k = i & 63;
        x[q] = row0 + m < n ? X[(row0 + m) * kIn + k] : 0.0f;
    }
    const int col = 32 * w + (lane_of() & 31);
    const float bn1 = p[kOffB1 + col], bn2 = p[kOffB2 + col], bn3 = p[kOffB3 + col], b4 = p[kOffB4];
    bf16_t w4[4];
#pragma unroll
    for (int j = 0; j < 4; j++) w4[j] = pk[kPkW4 + lane_of() + 64 * j];
    u16x8 b1[kIn / 16], b2[kHid / 16], b3[kHid / 16];
    load_frags<kIn>(pk + kPkF1, w, b1);
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const int i = threadIdx.x + q * kBlock, m = i >> 6, k = i & 63;
        xs[m * LDX + k] = row0 + m < n ? f2bf(x[q]) : (bf16_t)0;
    }
    lds_barrier();
    f32x16 acc[MT];
    mma_layer<MT, kIn>(xs, LDX, b1, acc);
    store_relu<MT>(acc, w, bn1, h0);
    lds_barrier();
    load_frags<kHid>(pk + kPkF2, w, b2);
    mma_layer<MT, kHid>(h0, LDA, b2, acc);
    store_relu<MT>(acc, w, bn2, h1);
    lds_barrier();
    load_frags<kHid>(pk + kPkF3, w, b3);
    mma_layer<MT, kHid>(h1, LDA, b3, acc);
    store_relu<MT>(acc, w, bn3, h0);
    lds_barrier();
    constexpr int PERW = R / kWaves;
    float y[PERW];
    head_rows<PERW>(h0, w, kWaves, w4, b4, y);
#pragma unroll
    for (int i = 0; i < PERW; i++) {
        const int m = w + i * kWaves;
        if (lane_of() == 0 && row0 + m < n) yhat[row0 + m] = y[i];
    }
}

// ------------------------------------------------------------------ training

// Forward and backward of rows [32 blockIdx.x, +32) of one minibatch of
// `batch` rows: row r is sample order[step * batch + r] (or r).
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void train_rows_kernel(const float *__restrict__ X, const float *__restrict__ Y,
                                                            const int32_t *__restrict__ order, long long step,
                                                            int batch, const State st, const TrainWs ws)
{
    constexpr int R = 32;
    __shared__ __attribute__((aligned(16))) bf16_t xs[R * LDX];
    __shared__ __attribute__((aligned(16))) bf16_t a1[R * LDA];
    __shared__ __attribute__((aligned(16))) bf16_t a2[R * LDA];
    __shared__ __attribute__((aligned(16))) bf16_t a3[R * LDA];
    __shared__ __attribute__((aligned(16))) bf16_t g3[R * LDA];
    __shared__ __attribute__((aligned(16))) bf16_t g2[R * LDA];
    __shared__ float tgt[R], dys[R], lss[R];
    const int bp = (batch + 31) / 32 * 32;
    const int row0 = blockIdx.x * R;
    const long long base = step * (long long)batch;
    const float *p = st.p;
    const bf16_t *pk = st.pk;
    const int w = wave_of();
    // the minibatch's rows first, then what every layer needs besides its
    // weights: with one block per CU nothing else hides their latency
    constexpr int PER = R * kIn / kBlock;
    const int k0 = threadIdx.x & 63;
    long long src[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const int r = row0 + w + q * kWaves;
        src[q] = r < batch ? (order ? order[base + r] : r) : -1;
    }
    float x[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) x[q] = src[q] >= 0 ? X[src[q] * kIn + k0] : 0.0f;
    float y0 = 0.0f;
    if (k0 < PER) {   // lane q of a wave loads the target of the wave's q-th row
        const int r = row0 + w + k0 * kWaves;
        if (r < batch) y0 = Y[order ? order[base + r] : r];
    }
    const int col = 32 * w + (lane_of() & 31);
    const float bn1 = p[kOffB1 + col], bn2 = p[kOffB2 + col], bn3 = p[kOffB3 + col], b4 = p[kOffB4];
    const bf16_t w4k = pk[kPkW4 + (threadIdx.x & (kHid - 1))];
    bf16_t w4[4];
#pragma unroll
    for (int j = 0; j < 4; j++) w4[j] = pk[kPkW4 + lane_of() + 64 * j];
    u16x8 b1[kIn / 16], b2[kHid / 16], b3[kHid / 16];
    load_frags<kIn>(pk + kPkF1, w, b1);
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const int m = w + q * kWaves;
        xs[m * LDX + k0] = src[q] >= 0 ? f2bf(x[q]) : (bf16_t)0;
    }
    if (k0 < PER) tgt[w + k0 * kWaves] = y0;
    lds_barrier();
    float *part = ws.part + (size_t)blockIdx.x * kPartStride;
    f32x16 acc[1];
    mma_layer<1, kIn>(xs, LDX, b1, acc);
    store_relu<1>(acc, w, bn1, a1, ws.aT[1], bp, row0);
    lds_barrier();
    load_frags<kHid>(pk + kPkF2, w, b2);
    mma_layer<1, kHid>(a1, LDA, b2, acc);
    // the backward products' weights take the registers of the forward ones
    load_frags<kHid>(pk + kPkB3, w, b2);
    store_relu<1>(acc, w, bn2, a2, ws.aT[2], bp, row0);
    lds_barrier();
    load_frags<kHid>(pk + kPkF3, w, b3);
    mma_layer<1, kHid>(a2, LDA, b3, acc);
    load_frags<kHid>(pk + kPkB2, w, b3);
    store_relu<1>(acc, w, bn3, a3);
    store_transposed(xs, LDX, kIn, ws.aT[0], bp, row0);
    lds_barrier();
    // head: dL/dy = clamp(y - t, -h, h) / batch for the Huber loss
    {
        constexpr int PERW = R / kWaves;
        float y[PERW];
        head_rows<PERW>(a3, w, kWaves, w4, b4, y);
        float yl = 0.0f;   // lane i: row w + 8 i
#pragma unroll
        for (int i = 0; i < PERW; i++) yl = lane_of() == i ? y[i] : yl;
        if (lane_of() < PERW) {
            const int m = w + lane_of() * kWaves;
            const bool ok = row0 + m < batch;
            const float e = yl - tgt[m];
            const float ae = fabsf(e);
            dys[m] = ok ? fminf(fmaxf(e, -kHuber), kHuber) / (float)batch : 0.0f;
            lss[m] = ok ? (ae <= kHuber ? 0.5f * e * e : kHuber * (ae - 0.5f * kHuber)) : 0.0f;
        }
    }
    lds_barrier();
    // delta of layer 3 (masked by a3 > 0) and the head gradients: the first
    // half of the threads sums a column of deltas each, the second half
    // stores it and sums the head's gradient
    {
        const int k = threadIdx.x & (kHid - 1);
        const float w4f = bf2f(w4k);
        const bool first = w < kWaves / 2;
        float sum = 0.0f;
        if (first) {
#pragma unroll
            for (int m = 0; m < R; m++) sum += bf2f(a3[m * LDA + k]) > 0.0f ? dys[m] * w4f : 0.0f;
        } else {
#pragma unroll
            for (int m0 = 0; m0 < R; m0 += 8) {
                u16x8 g;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    const float a = bf2f(a3[(m0 + i) * LDA + k]);
                    const float d = dys[m0 + i];
                    sum += a * d;
                    g[i] = f2bf(a > 0.0f ? d * w4f : 0.0f);
                    g3[(m0 + i) * LDA + k] = g[i];
                }
                *(u16x8 *)&ws.gT[2][(size_t)k * bp + row0 + m0] = g;
            }
        }
        part[(first ? kPartColsum + 2 * kHid : kPartW4) + k] = sum;
        if (threadIdx.x == 0 || threadIdx.x == 64) {
            const float *v = threadIdx.x == 0 ? dys : lss;
            float t = 0.0f;
#pragma unroll
            for (int m = 0; m < R; m++) t += v[m];
            part[threadIdx.x == 0 ? kPartB4 : kPartLoss] = t;
        }
    }
    lds_barrier();
    // delta of layer 2 = (g3 W3^T) masked by a2 > 0
    mma_layer<1, kHid>(g3, LDA, b2, acc);
    store_masked(acc[0], w, a2, g2, ws.gT[1], bp, row0, part + kPartColsum + kHid);
    lds_barrier();
    // delta of layer 1 = (g2 W2^T) masked by a1 > 0
    mma_layer<1, kHid>(g2, LDA, b3, acc);
    store_masked(acc[0], w, a1, nullptr, ws.gT[0], bp, row0, part + kPartColsum);
}

// Adam on one float32 master parameter with value pv and moments mv, vv;
// returns the new value
__device__ __forceinline__ float adam(const State &st, int i, float g, float pv, float mv, float vv, const Hyper &h,
                                      float c1, float c2)
{
    const float mi = h.b1 * mv + (1.0f - h.b1) * g;
    const float vi = h.b2 * vv + (1.0f - h.b2) * g * g;
    st.m[i] = mi;
    st.v[i] = vi;
    const float pi = pv - h.lr * (mi / c1) / (sqrtf(vi / c2) + h.eps);
    st.p[i] = pi;
    return pi;
}

__device__ __forceinline__ float adam(const State &st, int i, float g, const Hyper &h, float c1, float c2)
{
    return adam(st, i, g, st.p[i], st.m[i], st.v[i], h, c1, c2);
}

constexpr int kGradTiles = (kIn / 32) * 8 + 2 * 8 * 8;   // 32x32 tiles of gW1, gW2, gW3: 144
constexpr int kGradBlocks = kGradTiles + 5;              // then b1, b2, b3 and W4, and one block for b4 and the loss

// sum of part[b * kPartStride] over the nb blocks, in block order (eight loads in flight)
__device__ __forceinline__ float sum_parts(const float *part, int nb)
{
    float s = 0.0f;
    int b = 0;
    for (; b + 8 <= nb; b += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = part[(size_t)(b + i) * kPartStride];
#pragma unroll
        for (int i = 0; i < 8; i++) s += v[i];
    }
    for (; b < nb; b++) s += part[(size_t)b * kPartStride];
    return s;
}

// Weight gradients of one minibatch from the transposed activations and
// deltas (gW_l[i][j] = sum over rows of a_{l-1}[r][i] g_l[r][j]), then Adam
// (ADAM; `step` steps after the steps the state counts) or the gradient
// written flat into grads (!ADAM).  A block has one tile on a CU of its own:
// the work is a chain of loads and then of Adam's divisions and roots, so the
// first wave computes the tile and all four update a quarter of it each, with
// everything they read in flight before the products (12.6 us a step before,
// with one wave's loads and updates in turn; 8.6 us with every wave computing
// the tile).
constexpr int kGradBlock = 256;

template <bool ADAM>
__global__ __launch_bounds__(kGradBlock) void weight_grad_kernel(long long step, int batch, const State st,
                                                                 const TrainWs ws, float *__restrict__ grads,
                                                                 float *__restrict__ loss_out)
{
    const int bp = (batch + 31) / 32 * 32;
    const int lane = lane_of(), w = wave_of();
    Hyper h{};
    float t = 1.0f;
    if (ADAM) {
        h = *st.hyper;
        t = (float)(st.steps[0] + step + 1);
    }
    if (blockIdx.x < kGradTiles) {
        int tile = blockIdx.x;
        int layer, mt, nt, fan_in;
        if (tile < 16) {
            layer = 0; fan_in = kIn;
        } else {
            tile -= 16;
            layer = 1 + tile / 64;
            tile %= 64;
            fan_in = kHid;
        }
        mt = tile >> 3;
        nt = tile & 7;
        const bf16_t *AT = ws.aT[layer] + (size_t)(32 * mt + (lane & 31)) * bp + 8 * (lane >> 5);
        const bf16_t *GT = ws.gT[layer] + (size_t)(32 * nt + (lane & 31)) * bp + 8 * (lane >> 5);
        const int offW = layer == 0 ? kOffW1 : layer == 1 ? kOffW2 : kOffW3;
        const int pkF = layer == 0 ? kPkF1 : layer == 1 ? kPkF2 : kPkF3;
        const int pkB = layer == 1 ? kPkB2 : kPkB3;
        const int j = 32 * nt + (lane & 31);
        const int i0 = 32 * mt + acc_row(4 * w);   // this wave's four rows: elements 4 w ..
        const int idx0 = offW + i0 * kHid + j;
        __shared__ float s_tile[4][64][4];
        float pv[4], mv[4], vv[4], c1 = 1.0f, c2 = 1.0f;
        auto load_masters = [&]() {
            if (!ADAM) return;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                pv[e] = st.p[idx0 + e * kHid];
                mv[e] = st.m[idx0 + e * kHid];
                vv[e] = st.v[idx0 + e * kHid];
            }
        };
        if (w == 0) {
            f32x16 acc;
#pragma unroll
            for (int i = 0; i < 16; i++) acc[i] = 0.0f;
            const int ksteps = bp / 16;
            constexpr int KU = 16;   // k steps whose operands are in flight together
            u16x8 a[KU], b[KU];
            auto load = [&](int ks) {
#pragma unroll
                for (int q = 0; q < KU; q++) {
                    if (ks + q >= ksteps) continue;
                    a[q] = *(const u16x8 *)(AT + 16 * (ks + q));
                    b[q] = *(const u16x8 *)(GT + 16 * (ks + q));
                }
            };
            load(0);
            load_masters();
            for (int ks = 0; ks < ksteps; ks += KU) {
#pragma unroll
                for (int q = 0; q < KU; q++) {
                    if (ks + q >= ksteps) continue;
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[q]),
                                                                  __builtin_bit_cast(bf16x8, b[q]), acc, 0, 0, 0);
                }
                load(ks + KU);
            }
#pragma unroll
            for (int i = 0; i < 16; i++) s_tile[i >> 2][lane][i & 3] = acc[i];
        } else {
            load_masters();
        }
        if (ADAM) {
            c1 = 1.0f - powf(h.b1, t);
            c2 = 1.0f - powf(h.b2, t);
        }
        lds_barrier();
        float g[4];
#pragma unroll
        for (int e = 0; e < 4; e++) g[e] = s_tile[w][lane][e];
        if (!ADAM) {
#pragma unroll
            for (int e = 0; e < 4; e++) grads[idx0 + e * kHid] = g[e];
            return;
        }
        // four consecutive rows i: one 8-byte store of the forward packing
        uint16_t wb[4];
#pragma unroll
        for (int e = 0; e < 4; e++) wb[e] = f2bf(adam(st, idx0 + e * kHid, g[e], pv[e], mv[e], vv[e], h, c1, c2));
        *(uint2 *)&st.pk[pkF + frag_off(i0, j, fan_in)] =
            make_uint2((uint32_t)wb[0] | (uint32_t)wb[1] << 16, (uint32_t)wb[2] | (uint32_t)wb[3] << 16);
        if (layer > 0) {
#pragma unroll
            for (int e = 0; e < 4; e++) st.pk[pkB + frag_off(j, i0 + e, kHid)] = wb[e];
        }
        return;
    }
    // biases, W4 and b4 from the per-block partials (summed in block order)
    const int nb = bp / 32;
    const float c1 = ADAM ? 1.0f - powf(h.b1, t) : 1.0f, c2 = ADAM ? 1.0f - powf(h.b2, t) : 1.0f;
    const int l = blockIdx.x - kGradTiles;
    static_assert(kGradBlock == kHid, "a thread per column");
    if (l < 4) {
        const int off = (l == 0 ? kOffB1 : l == 1 ? kOffB2 : l == 2 ? kOffB3 : kOffW4) + (int)threadIdx.x;
        const float s = sum_parts(ws.part + (l < 3 ? kPartColsum + l * kHid : kPartW4) + threadIdx.x, nb);
        if (ADAM) {
            const float wn = adam(st, off, s, h, c1, c2);
            if (l == 3) st.pk[kPkW4 + threadIdx.x] = f2bf(wn);
        } else {
            grads[off] = s;
        }
    } else if (threadIdx.x == 0) {
        const float s = sum_parts(ws.part + kPartB4, nb);
        if (ADAM) adam(st, kOffB4, s, h, c1, c2);
        else grads[kOffB4] = s;
    } else if (threadIdx.x == 64 && loss_out) {
        loss_out[step] = sum_parts(ws.part + kPartLoss, nb) / (float)batch;
    }
}

__global__ void advance_kernel(long long *steps, long long n) { steps[0] += n; }

__global__ void begin_call_kernel(Hyper *hyper, float lr) { *hyper = Hyper{lr, 0.9f, 0.999f, 1e-8f}; }

// bf16 packings of the weights from the float32 master copy
__global__ void pack_kernel(const float *__restrict__ p, bf16_t *__restrict__ pk)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kIn * kHid) {
        pk[kPkF1 + frag_off(i / kHid, i % kHid, kIn)] = f2bf(p[kOffW1 + i]);
    } else if (i < kIn * kHid + 2 * kHid * kHid) {
        const int l = (i - kIn * kHid) / (kHid * kHid);
        const int q = (i - kIn * kHid) % (kHid * kHid);
        const int r = q / kHid, c = q % kHid;
        const bf16_t wb = f2bf(p[(l == 0 ? kOffW2 : kOffW3) + q]);
        pk[(l == 0 ? kPkF2 : kPkF3) + frag_off(r, c, kHid)] = wb;
        pk[(l == 0 ? kPkB2 : kPkB3) + frag_off(c, r, kHid)] = wb;
    } else if (i < kIn * kHid + 2 * kHid * kHid + kHid) {
        const int k = i - kIn * kHid - 2 * kHid * kHid;
        pk[kPkW4 + k] = f2bf(p[kOffW4 + k]);
    }
}

}  // namespace esc

using namespace esc;

struct esc_mlp {
    int device = 0;
    int num_cus = 0;
    char *state = nullptr;   // caller-owned, kStateBytes
    State st{};
    hipStream_t cap = nullptr;   // private stream for state transfers
};

namespace {

int hipchk(hipError_t e, const char *what) { return e == hipSuccess ? ESC_OK : hip_fail(e, what); }

int check_mlp(const esc_mlp *m)
{
    if (!m) return fail(ESC_ERR_INVALID, "null mlp handle");
    return set_device(m->device);
}

int check_ws(const void *ws, size_t bytes, int batch)
{
    if (!ws || ((uintptr_t)ws & 255)) return fail(ESC_ERR_ALIGN, "workspace must be non-null and 256-byte aligned");
    const size_t need = train_ws_bytes(batch, nullptr, nullptr);
    if (bytes < need) return fail(ESC_ERR_OOM, "workspace of %zu bytes, %zu needed for %d rows", bytes, need, batch);
    return ESC_OK;
}

// 64-bit FNV-1a over a byte range (checkpoint integrity)
uint64_t fnv1a(const void *data, size_t n, uint64_t h)
{
    const unsigned char *b = (const unsigned char *)data;
    for (size_t i = 0; i < n; i++) {
        h ^= b[i];
        h *= 0x100000001b3ull;
    }
    return h;
}

constexpr char kMagic[8] = {'E', 'S', 'C', 'M', 'L', 'P', '0', '1'};
constexpr uint32_t kFileVersion = 1;

struct FileHeader {
    char magic[8];
    uint32_t version;
    uint32_t nparams;
    int64_t step;
    uint64_t checksum;   // FNV-1a of params, m and v
};

}  // namespace

extern "C" {

size_t esc_mlp_state_bytes(void) { return kStateBytes; }

size_t esc_mlp_workspace_bytes(int batch)
{
    if (batch < 1 || batch > kMaxBatch) return 0;
    return train_ws_bytes(batch, nullptr, nullptr);
}

int esc_mlp_create(esc_ctx *ctx, void *dev_state, size_t state_bytes, esc_mlp **out)
{
    if (!ctx || !out) return fail(ESC_ERR_INVALID, "null argument");
    if (!dev_state || ((uintptr_t)dev_state & 255)) return fail(ESC_ERR_ALIGN, "state must be 256-byte aligned");
    if (state_bytes < kStateBytes) return fail(ESC_ERR_OOM, "state of %zu bytes, %zu needed", state_bytes, kStateBytes);
    if (int rc0 = set_device(ctx->device)) return rc0;
    esc_mlp *m = new (std::nothrow) esc_mlp;
    if (!m) return fail(ESC_ERR_OOM, "out of host memory");
    m->device = ctx->device;
    m->num_cus = ctx->num_cus;
    m->state = (char *)dev_state;
    m->st = State{(float *)(m->state + kStP), (float *)(m->state + kStM), (float *)(m->state + kStV),
                  (long long *)(m->state + kStSteps), (Hyper *)(m->state + kStHyper), (bf16_t *)(m->state + kStPack)};
    hipError_t e = hipStreamCreateWithFlags(&m->cap, hipStreamNonBlocking);
    if (e != hipSuccess) { delete m; return hip_fail(e, "stream"); }
    std::vector<float> z(kNParams, 0.0f);
    int rc = esc_mlp_set_params(m, z.data());
    if (rc) { esc_mlp_destroy(m); return rc; }
    *out = m;
    return ESC_OK;
}

int esc_mlp_destroy(esc_mlp *m)
{
    if (!m) return ESC_OK;
    (void)set_device(m->device);
    if (m->cap) (void)hipStreamDestroy(m->cap);
    delete m;
    return ESC_OK;
}

int esc_mlp_set_state(esc_mlp *m, const float *params, const float *adam_m, const float *adam_v, int64_t step)
{
    int rc = check_mlp(m);
    if (rc) return rc;
    if (!params || step < 0) return fail(ESC_ERR_INVALID, "null parameters or negative step");
    hipStream_t s = m->cap;
    if ((rc = hipchk(hipMemcpyAsync(m->st.p, params, kNParams * 4, hipMemcpyHostToDevice, s), "upload"))) return rc;
    if (adam_m) rc = hipchk(hipMemcpyAsync(m->st.m, adam_m, kNParams * 4, hipMemcpyHostToDevice, s), "upload");
    else rc = hipchk(hipMemsetAsync(m->st.m, 0, kNParams * 4, s), "memset");
    if (rc) return rc;
    if (adam_v) rc = hipchk(hipMemcpyAsync(m->st.v, adam_v, kNParams * 4, hipMemcpyHostToDevice, s), "upload");
    else rc = hipchk(hipMemsetAsync(m->st.v, 0, kNParams * 4, s), "memset");
    if (rc) return rc;
    const long long steps[2] = {(long long)step, 0};
    if ((rc = hipchk(hipMemcpyAsync(m->st.steps, steps, sizeof steps, hipMemcpyHostToDevice, s), "upload"))) return rc;
    constexpr int kPackItems = kIn * kHid + 2 * kHid * kHid + kHid;
    hipLaunchKernelGGL(pack_kernel, dim3((kPackItems + 255) / 256), dim3(256), 0, s, m->st.p, m->st.pk);
    return hipchk(hipStreamSynchronize(s), "sync");
}

int esc_mlp_set_params(esc_mlp *m, const float *host_params)
{
    return esc_mlp_set_state(m, host_params, nullptr, nullptr, 0);
}

int esc_mlp_get_state(esc_mlp *m, float *params, float *adam_m, float *adam_v, int64_t *step)
{
    int rc = check_mlp(m);
    if (rc) return rc;
    hipStream_t s = m->cap;
    if (params && (rc = hipchk(hipMemcpyAsync(params, m->st.p, kNParams * 4, hipMemcpyDeviceToHost, s), "download")))
        return rc;
    if (adam_m && (rc = hipchk(hipMemcpyAsync(adam_m, m->st.m, kNParams * 4, hipMemcpyDeviceToHost, s), "download")))
        return rc;
    if (adam_v && (rc = hipchk(hipMemcpyAsync(adam_v, m->st.v, kNParams * 4, hipMemcpyDeviceToHost, s), "download")))
        return rc;
    long long steps[2] = {0, 0};
    if ((rc = hipchk(hipMemcpyAsync(steps, m->st.steps, sizeof steps, hipMemcpyDeviceToHost, s), "download")))
        return rc;
    if ((rc = hipchk(hipStreamSynchronize(s), "sync"))) return rc;
    if (step) *step = steps[0];
    return ESC_OK;
}

int esc_mlp_get_params(esc_mlp *m, float *host_params)
{
    if (!host_params) return fail(ESC_ERR_INVALID, "null output");
    return esc_mlp_get_state(m, host_params, nullptr, nullptr, nullptr);
}

int esc_mlp_save(esc_mlp *m, const char *path)
{
    if (!path) return fail(ESC_ERR_INVALID, "null path");
    std::vector<float> buf(3 * (size_t)kNParams);
    int64_t step = 0;
    int rc = esc_mlp_get_state(m, buf.data(), buf.data() + kNParams, buf.data() + 2 * kNParams, &step);
    if (rc) return rc;
    FileHeader h{};
    memcpy(h.magic, kMagic, 8);
    h.version = kFileVersion;
    h.nparams = kNParams;
    h.step = step;
    h.checksum = fnv1a(buf.data(), buf.size() * 4, 0xcbf29ce484222325ull);
    FILE *f = fopen(path, "wb");
    if (!f) return fail(ESC_ERR_INVALID, "cannot open %s for writing", path);
    const bool ok = fwrite(&h, sizeof h, 1, f) == 1 && fwrite(buf.data(), 4, buf.size(), f) == buf.size();
    const bool closed = fclose(f) == 0;
    if (!ok || !closed) return fail(ESC_ERR_INVALID, "writing %s failed", path);
    return ESC_OK;
}

int esc_mlp_load(esc_mlp *m, const char *path)
{
    if (!path) return fail(ESC_ERR_INVALID, "null path");
    int rc = check_mlp(m);
    if (rc) return rc;
    FILE *f = fopen(path, "rb");
    if (!f) return fail(ESC_ERR_INVALID, "cannot open %s", path);
    FileHeader h{};
    std::vector<float> buf(3 * (size_t)kNParams);
    const bool ok = fread(&h, sizeof h, 1, f) == 1 && fread(buf.data(), 4, buf.size(), f) == buf.size();
    char extra;
    const bool at_end = fread(&extra, 1, 1, f) == 0;
    fclose(f);
    if (!ok || !at_end) return fail(ESC_ERR_INVALID, "%s: wrong size for an estimator checkpoint", path);
    if (memcmp(h.magic, kMagic, 8) != 0) return fail(ESC_ERR_INVALID, "%s: not an estimator checkpoint", path);
    if (h.version != kFileVersion || h.nparams != (uint32_t)kNParams)
        return fail(ESC_ERR_INVALID, "%s: version %u with %u parameters, expected %u with %d", path, h.version,
                    h.nparams, kFileVersion, kNParams);
    if (h.step < 0) return fail(ESC_ERR_INVALID, "%s: negative step count", path);
    if (fnv1a(buf.data(), buf.size() * 4, 0xcbf29ce484222325ull) != h.checksum)
        return fail(ESC_ERR_INVALID, "%s: checksum mismatch", path);
    return esc_mlp_set_state(m, buf.data(), buf.data() + kNParams, buf.data() + 2 * kNParams, h.step);
}

int esc_mlp_predict(esc_mlp *m, const float *dev_x, int64_t n, float *dev_yhat, void *stream)
{
    int rc = check_mlp(m);
    if (rc) return rc;
    if (n < 0 || (n > 0 && (!dev_x || !dev_yhat))) return fail(ESC_ERR_INVALID, "bad arguments");
    if (n == 0) return ESC_OK;
    hipStream_t s = (hipStream_t)stream;
    // 64 rows a block read each weight half as often, but every 64 rows a CU
    // begun take the time of all: 32 rows are faster for up to three such
    // blocks a CU and for a fifth (us by 32 and by 64: 4,096 rows 6.6 and 9.4,
    // 16,384 9.6 and 9.6, 18,000 12.0 and 14.0, 24,576 12.6 and 14.2, 28,000
    // 15.5 and 14.3, 36,000 18.9 and 20.6, 49,152 23.2 and 21.0, 262,144 115
    // and 107)
    const int64_t tiles = (n + 32ll * m->num_cus - 1) / (32ll * m->num_cus);
    if (tiles <= 3 || tiles == 5)
        hipLaunchKernelGGL(forward_kernel<1>, dim3((unsigned)((n + 31) / 32)), dim3(kBlock), 0, s, dev_x, n, m->st.p,
                           m->st.pk, dev_yhat);
    else
        hipLaunchKernelGGL(forward_kernel<2>, dim3((unsigned)((n + 63) / 64)), dim3(kBlock), 0, s, dev_x, n, m->st.p,
                           m->st.pk, dev_yhat);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ESC_OK : hip_fail(e, "predict launch");
}

int esc_mlp_gradients(esc_mlp *m, const float *dev_x, const float *dev_y, int64_t n, float *dev_grads,
                      void *dev_ws, size_t ws_bytes, void *stream)
{
    int rc = check_mlp(m);
    if (rc) return rc;
    if (n < 1 || n > kMaxBatch || !dev_x || !dev_y || !dev_grads)
        return fail(ESC_ERR_INVALID, "need 1 <= n <= %d and non-null buffers", kMaxBatch);
    if ((rc = check_ws(dev_ws, ws_bytes, (int)n))) return rc;
    hipStream_t s = (hipStream_t)stream;
    TrainWs ws;
    train_ws_bytes((int)n, &ws, (char *)dev_ws);
    const int nb = (int)((n + 31) / 32);
    hipLaunchKernelGGL(train_rows_kernel, dim3(nb), dim3(kBlock), 0, s, dev_x, dev_y, nullptr, 0ll, (int)n, m->st,
                       ws);
    hipLaunchKernelGGL(weight_grad_kernel<false>, dim3(kGradBlocks), dim3(kGradBlock), 0, s, 0ll, (int)n, m->st, ws, dev_grads,
                       nullptr);
    return hipchk(hipStreamSynchronize(s), "sync");
}

int esc_mlp_train(esc_mlp *m, const float *dev_x, const float *dev_y, const int32_t *dev_order, int64_t steps,
                  int batch, float lr, void *dev_ws, size_t ws_bytes, void *stream, float *dev_loss)
{
    int rc = check_mlp(m);
    if (rc) return rc;
    if (steps < 0 || batch < 1 || batch > kMaxBatch || !dev_x || !dev_y || !dev_order || !(lr > 0.0f))
        return fail(ESC_ERR_INVALID, "bad training arguments");
    if ((rc = check_ws(dev_ws, ws_bytes, batch))) return rc;
    if (steps == 0) return ESC_OK;
    hipStream_t s = (hipStream_t)stream;
    TrainWs ws;
    train_ws_bytes(batch, &ws, (char *)dev_ws);
    hipLaunchKernelGGL(begin_call_kernel, dim3(1), dim3(1), 0, s, m->st.hyper, lr);
    // two launches per step, in stream order; each knows its step, and the
    // count of steps in the state moves on once, behind the last
    const int nb = (batch + 31) / 32;
    hipError_t e = hipSuccess;
    int64_t done = 0;
    for (; done < steps && e == hipSuccess; done++) {
        hipLaunchKernelGGL(train_rows_kernel, dim3(nb), dim3(kBlock), 0, s, dev_x, dev_y, dev_order, (long long)done,
                           batch, m->st, ws);
        hipLaunchKernelGGL(weight_grad_kernel<true>, dim3(kGradBlocks), dim3(kGradBlock), 0, s, (long long)done, batch, m->st,
                           ws, nullptr, dev_loss);
        e = hipGetLastError();
    }
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(1), 0, s, m->st.steps, (long long)done);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e == hipSuccess ? ESC_OK : hip_fail(e, "training");
}

}  // extern "C"
