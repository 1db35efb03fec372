// Learned weight proposer (form F3): front-gap features, a small MLP
// (D -> 128 -> 128 -> 1, exact-erf GELU, bf16 weights, fp32 activations and
// accumulation), its mean binary cross-entropy gradient, Adam, top-k
// selection and the labels "this weight vector produced a new non-dominated
// point".  The paper has no learned component; the proposer chooses which
// scalarisation weight vectors (Eq. 7) the sampler runs next.
//
// Parameter layout (flat): W1 [H][D], b1 [H], W2 [H][H], b2 [H], w3 [H], b3.

#include <cmath>

#include "radix.hpp"

namespace qaia {
namespace {

constexpr int kH = 128;
constexpr int kB = 256;
constexpr int kMaxD = 16;

struct ParamOffsets {
    int64_t W1, b1, W2, b2, w3, b3, total;
};
__host__ __device__ inline ParamOffsets offsets(int D) {
    ParamOffsets o;
    o.W1 = 0;
    o.b1 = o.W1 + (int64_t)kH * D;
    o.W2 = o.b1 + kH;
    o.b2 = o.W2 + (int64_t)kH * kH;
    o.w3 = o.b2 + kH;
    o.b3 = o.w3 + kH;
    o.total = o.b3 + 1;
    return o;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round half to even (finite values)
    return (uint16_t)(u >> 16);
}
// 1 + erf(z / sqrt 2) is evaluated as erfc(-z / sqrt 2): for negative z the
// sum would cancel (at z = -5 it is 1.5e-6, below the float32 spacing of the
// erf value near -1), the complementary function keeps full relative accuracy.
__device__ __forceinline__ float gelu(float z) { return 0.5f * z * erfcf(-z * 0.70710678118654752f); }
__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * erfcf(-z * 0.70710678118654752f) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ---------------------------------------------------------------- MLP passes
//
// One block of sixteen waves handles 32 samples.  Layer 1 (D -> 128, tiny) and
// the activations run on the vector units; the 128 x 128 contractions run on
// the matrix cores as fp32 32x32x2 MFMAs (the bf16 weights widen exactly to
// fp32, so activations and accumulation stay fp32):
//   forward : Z2 = A1 W2^T, waves 0 .. 3 take 32 units each;
//   backward: dZ1 = dZ2 W2 (a wave per 32 hidden units), and
//             dW2 = dZ2^T A1 (a wave per tile of 32 units x 32 columns).
// For every MFMA the A and B fragments of a lane come from the same k
// position (k = 2t + lane / 32), which pairs them for any internal k order.
// Accumulator slot i of lane l holds row (i/4)*8 + (l/32)*4 + i%4, column l%32.
// Training writes the block's gradient contribution (every parameter) to
// partial[block]; the blocks are summed in a fixed order.
//
// A batch of a few hundred samples leaves most of the chip idle and lasts one
// block's chain, so that is kept short: sixteen waves share the activations
// (some 60 instructions each, two per sample and unit in training), and with
// Q = 4 four blocks repeat the forward part of a tile and take a quarter of the
// hidden units' and of the columns' gradients each.  One 32-sample tile of
// twelve inputs in training: 29 us with four waves and no split, now 15.
constexpr int kS = 32;          // samples per block
constexpr int kP = kH + 2;      // LDS pitch (floats) of the 128-wide tiles: a 32-lane strided read and its
                                // neighbour column fall on disjoint banks
constexpr int kT = 1024;

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int acc_row(int half, int i) { return (i >> 2) * 8 + half * 4 + (i & 3); }

template <bool TRAIN, int Q>
__global__ __launch_bounds__(kT) void mlp_tile_kernel(const uint16_t *__restrict__ P, int D,
                                                      const float *__restrict__ X, int64_t N,
                                                      const float *__restrict__ y, float *__restrict__ logits,
                                                      float *__restrict__ partial) {
    __shared__ float w2[kH * kP];          // W2[u][h] at u * kP + h
    __shared__ float w1[kH][kMaxD + 1];
    __shared__ float xs[kS][kMaxD + 1];
    __shared__ float a1[kS * kP];          // A1[s][h]
    __shared__ float z2[kS * kP];          // Z2[s][u], then dZ2
    __shared__ float a2[TRAIN ? kS * kP : 1];   // gelu(Z2)
    __shared__ float g2[TRAIN ? kS * kP : 1];   // gelu'(Z2)
    __shared__ float g1[TRAIN ? kS * kP : 1];   // gelu'(z1)[s][h], then dZ1[s][h], of this block's h
    __shared__ float dz3[kS];
    const ParamOffsets o = offsets(D);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, lr = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), q = Q == 1 ? 0 : blockIdx.y;
    const int64_t s0 = (int64_t)blockIdx.x * kS;
    const int ns = (int)(N - s0 < kS ? N - s0 : kS);
    if ((((uintptr_t)(P + o.W2)) & 15) == 0) {
        // eight bf16 weights per 16-byte load (W2 starts at 128 (D + 1) elements)
        const uint4 *src = (const uint4 *)(P + o.W2);
#pragma unroll
        for (int i = tid; i < kH * kH / 8; i += kT) {
            const uint4 w = src[i];
            float *dst = w2 + ((i * 8) >> 7) * kP + ((i * 8) & (kH - 1));
            const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dst[2 * e] = __uint_as_float(u[e] << 16);
                dst[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
            }
        }
    } else {
        for (int i = tid; i < kH * kH; i += kT) w2[(i >> 7) * kP + (i & (kH - 1))] = bf16_to_f32(P[o.W2 + i]);
    }
    for (int i = tid; i < kH * kMaxD; i += kT) {
        const int h = i / kMaxD, d = i % kMaxD;
        w1[h][d] = d < D ? bf16_to_f32(P[o.W1 + (int64_t)h * D + d]) : 0.0f;
    }
    if (tid < kS * kMaxD) {
        const int s = tid / kMaxD, d = tid % kMaxD;
        xs[s][d] = (s < ns && d < D) ? X[(s0 + s) * D + d] : 0.0f;
    }
    float b1v[4], b2v[4], w3v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        b1v[j] = bf16_to_f32(P[o.b1 + 32 * j + (tid >> 5)]);
        b2v[j] = bf16_to_f32(P[o.b2 + 32 * j + lr]);
        w3v[j] = bf16_to_f32(P[o.w3 + 32 * j + lr]);
    }
    const float b3 = bf16_to_f32(P[o.b3]);
    const int sr = 2 * wave + half;  // the sample of this half wave from layer 2 on
    float yv = 0.0f;
    if constexpr (TRAIN) yv = sr < ns ? y[s0 + sr] : 0.0f;
    __syncthreads();
    // layer 1: thread t takes sample t % 32 and hidden units t / 32 + 32 j
    {
        const int s = tid & (kS - 1), hg = tid >> 5;
        float z[4] = {b1v[0], b1v[1], b1v[2], b1v[3]};
        for (int d = 0; d < D; ++d) {
            const float x = xs[s][d];
#pragma unroll
            for (int j = 0; j < 4; ++j) z[j] = fmaf(w1[32 * j + hg][d], x, z[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a1[s * kP + 32 * j + hg] = gelu(z[j]);
            if constexpr (TRAIN)
                if (Q == 1 || j == q) g1[s * kP + 32 * j + hg] = gelu_grad(z[j]);
        }
    }
    __syncthreads();
    // layer 2 on the matrix cores: 32 units per wave
    if (wave < 4) {
        const int u = wave * 32 + lr;
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll 16
        for (int t = 0; t < kH / 2; ++t) {
            const int k = 2 * t + half;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[lr * kP + k], w2[u * kP + k], acc, 0, 0, 0);
        }
        const float b2u = wave == 0 ? b2v[0] : wave == 1 ? b2v[1] : wave == 2 ? b2v[2] : b2v[3];
#pragma unroll
        for (int i = 0; i < 16; ++i) z2[acc_row(half, i) * kP + u] = acc[i] + b2u;
    }
    __syncthreads();
    // head: half a wave per sample, summed over the 32 lanes of each unit tile,
    // then over the four tiles in a fixed order
    {
        float z[4], a[4], part[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            z[j] = z2[sr * kP + 32 * j + lr];
            a[j] = gelu(z[j]);
            part[j] = fmaf(w3v[j], a[j], __shfl_xor(w3v[j] * a[j], 16, 64));
        }
        for (int off = 8; off > 0; off >>= 1)
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j] += __shfl_xor(part[j], off, 64);
        // of the first lane: the fused first level makes the upper sixteen's sums other ones
        const float lg = __shfl(b3 + ((part[0] + part[1]) + (part[2] + part[3])), lane & 32, 64);
        if (lr == 0 && sr < ns && logits && q == 0) logits[s0 + sr] = lg;
        if constexpr (!TRAIN) return;
        // dZ2 = dz3 w3 gelu'(z2)
        const float d3 = sr < ns ? (1.0f / (1.0f + expf(-lg)) - yv) / (float)N : 0.0f;
        if (lr == 0) dz3[sr] = d3;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float g = gelu_grad(z[j]);
            g2[sr * kP + 32 * j + lr] = g;
            z2[sr * kP + 32 * j + lr] = d3 * w3v[j] * g;
            a2[sr * kP + 32 * j + lr] = a[j];
        }
    }
    __syncthreads();
    float *pg = partial + (int64_t)blockIdx.x * o.total;
    // gb2[u] = sum_s dZ2, gw3[u] = sum_s dz3 a2: waves 4 .. (their SIMDs' matrix work is elsewhere or waits)
    if (wave >= 4 && wave < 4 + (Q == 1 ? 4 : 1)) {
        const int j = q + wave - 4, u = 32 * j + lr;
        const float w3u = j == 0 ? w3v[0] : j == 1 ? w3v[1] : j == 2 ? w3v[2] : w3v[3];
        float gb2 = 0.0f, gw3 = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int s = acc_row(half, i);
            gb2 = fmaf(dz3[s] * w3u, g2[s * kP + u], gb2);
            gw3 = fmaf(dz3[s], a2[s * kP + u], gw3);
        }
        gb2 += __shfl_xor(gb2, 32, 64);
        gw3 += __shfl_xor(gw3, 32, 64);
        if (half == 0) {
            pg[o.b2 + u] = gb2;
            pg[o.w3 + u] = gw3;
        }
    }
    if (tid == 8 * 64 && q == 0) {
        float g3 = 0.0f;
        for (int s = 0; s < kS; ++s) g3 += dz3[s];
        pg[o.b3] = g3;
    }
    // dZ1 = (dZ2 W2) * gelu'(z1)
    if (wave < (Q == 1 ? 4 : 1)) {
        const int h = 32 * (q + wave) + lr;
        f32x16 d;
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = 0.0f;
#pragma unroll 16
        for (int t = 0; t < kH / 2; ++t) {
            const int k = 2 * t + half;  // the unit index u
            d = __builtin_amdgcn_mfma_f32_32x32x2f32(z2[lr * kP + k], w2[k * kP + h], d, 0, 0, 0);
        }
        float gb1 = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int s = acc_row(half, i);
            const float v = g1[s * kP + h];
            g1[s * kP + h] = d[i] * v;
            gb1 = fmaf(d[i], v, gb1);
        }
        gb1 += __shfl_xor(gb1, 32, 64);
        if (half == 0) pg[o.b1 + h] = gb1;
    }
    // dW2 = dZ2^T A1: a tile of rows u and columns h per wave, k = sample.  With
    // Q = 4 the tiles go to waves 1, 2, 3 and 5: wave 0's SIMD has the longer chain of dZ1
    {
        const int r = Q == 1 ? wave & 3 : wave == 5 ? 3 : wave - 1, c = Q == 1 ? wave >> 2 : q;
        if (Q == 1 || (wave >= 1 && wave <= 5 && wave != 4)) {
            f32x16 g;
#pragma unroll
            for (int i = 0; i < 16; ++i) g[i] = 0.0f;
#pragma unroll
            for (int t = 0; t < kS / 2; ++t) {
                const int s = 2 * t + half;
                g = __builtin_amdgcn_mfma_f32_32x32x2f32(z2[s * kP + r * 32 + lr], a1[s * kP + c * 32 + lr], g, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) pg[o.W2 + (int64_t)(r * 32 + acc_row(half, i)) * kH + c * 32 + lr] = g[i];
        }
    }
    __syncthreads();
    // dW1[h][d] = sum_s dZ1[s][h] x[s][d]: a thread per entry
    for (int i = tid; i < kH / Q * kMaxD; i += kT) {
        const int h = kH / Q * q + i / kMaxD, d = i % kMaxD;
        float g = 0.0f;
#pragma unroll 8
        for (int s = 0; s < kS; ++s) g = fmaf(g1[s * kP + h], xs[s][d], g);
        if (d < D) pg[o.W1 + (int64_t)h * D + d] = g;
    }
}

// Forward of many samples: one wave takes 32 samples through the whole network
// and keeps them in registers.  The operands of layer 2 are the other way round
// (rows = units, columns = samples), so lane l holds sample l % 32: it computes
// the hidden unit that its half contributes to the next MFMA itself, k by k, and
// the four unit tiles take it at once (four accumulators; no layer-1 tile in
// LDS, no barrier).  The 16 units of a lane's accumulator are summed in the
// order of the other kernel's shuffles (unit bits 4, 3, 2, 1, 0), four of the
// five levels of them in the lane.  Weights lie in LDS widened, W2 as
// [k parity][k / 8][unit][4]: one 16-byte read per four MFMAs, conflict-free
// when read and, with the pitch of 516, when filled along k.
// Bound by the vector unit: 256 gelus of some 57 instructions per sample, 28 us
// for 65 536 samples if nothing else ran; the MFMAs lie between them.  That many
// samples of twelve inputs: 123 to 133 us with a block of four waves per 32, now 46 to 48.
constexpr int kRWaves = 8;
constexpr int kW2Pitch = 4 * kH + 4;
constexpr int kW2Parity = 16 * kW2Pitch + 16;

template <int G>  // groups of four inputs
__global__ __launch_bounds__(64 * kRWaves) void mlp_rows_kernel(const uint16_t *__restrict__ P, int D,
                                                                const float *__restrict__ X, int64_t N,
                                                                float *__restrict__ logits) {
    __shared__ __align__(16) float w2[2 * kW2Parity];
    __shared__ __align__(16) float w1[kH * 4 * G];
    __shared__ __align__(16) float b1[2 * kH / 2], b2[kH], w3[kH];
    const ParamOffsets o = offsets(D);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, lr = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool wide = (((uintptr_t)(P + o.W2)) & 15) == 0;  // W2 starts at 128 (D + 1) elements
    for (int i = tid; i < kH * kH / 8; i += 64 * kRWaves) {
        const int u = i >> 4, c = i & 15;  // eight weights k = 8c .. of unit u
        uint4 w;
        if (wide) {
            w = ((const uint4 *)(P + o.W2))[i];
        } else {
            const uint16_t *q = P + o.W2 + 8 * i;
            w = make_uint4(q[0] | (uint32_t)q[1] << 16, q[2] | (uint32_t)q[3] << 16, q[4] | (uint32_t)q[5] << 16,
                           q[6] | (uint32_t)q[7] << 16);
        }
        float *dst = w2 + c * kW2Pitch + 4 * u;
        *(float4 *)dst = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.y << 16),
                                     __uint_as_float(w.z << 16), __uint_as_float(w.w << 16));
        *(float4 *)(dst + kW2Parity) =
            make_float4(__uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y & 0xFFFF0000u),
                        __uint_as_float(w.z & 0xFFFF0000u), __uint_as_float(w.w & 0xFFFF0000u));
    }
    for (int i = tid; i < kH * 4 * G; i += 64 * kRWaves) {
        const int h = i / (4 * G), d = i % (4 * G);
        w1[i] = d < D ? bf16_to_f32(P[o.W1 + (int64_t)h * D + d]) : 0.0f;
    }
    if (tid < kH) {
        b1[(tid & 1) * (kH / 2) + (tid >> 1)] = bf16_to_f32(P[o.b1 + tid]);
        b2[tid] = bf16_to_f32(P[o.b2 + tid]);
        w3[tid] = bf16_to_f32(P[o.w3 + tid]);
    }
    const float b3 = bf16_to_f32(P[o.b3]);
    __syncthreads();
    const float *wl = w2 + half * kW2Parity + 4 * lr;
    const float *w1l = w1 + half * 4 * G;
    const float *b1l = b1 + half * (kH / 2);
    for (int64_t tile = blockIdx.x + (int64_t)gridDim.x * wave; tile * kS < N; tile += (int64_t)gridDim.x * kRWaves) {
        const int64_t s = tile * kS + lr;
        float x[4 * G];
#pragma unroll
        for (int d = 0; d < 4 * G; ++d) {  // 0 * -0 + z is z for every z
            x[d] = X[(s < N ? s : N - 1) * D + (d < D ? d : D - 1)];
            if (d >= D) x[d] = -0.0f;
        }
        auto hidden = [&](int c, float *a) {
            const float4 bb = *(const float4 *)(b1l + 4 * c);
            const float zb[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float z = zb[e];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float4 w = *(const float4 *)(w1l + (8 * c + 2 * e) * 4 * G + 4 * g);
                    z = fmaf(w.x, x[4 * g], z);
                    z = fmaf(w.y, x[4 * g + 1], z);
                    z = fmaf(w.z, x[4 * g + 2], z);
                    z = fmaf(w.w, x[4 * g + 3], z);
                }
                a[e] = gelu(z);
            }
        };
        f32x16 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[j][i] = 0.0f;
        float a[4];
        hidden(0, a);
#pragma unroll 1
        for (int c = 0; c < 16; ++c) {
            float next[4];
            float4 w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = *(const float4 *)(wl + c * kW2Pitch + 128 * j);
            hidden((c + 1) & 15, next);  // the last one is not used
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float we = e == 0 ? w[j].x : e == 1 ? w[j].y : e == 2 ? w[j].z : w[j].w;
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(we, a[e], acc[j], 0, 0, 0);
                }
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an MFMA takes 64 cycles,
                __builtin_amdgcn_sched_group_barrier(0x002, 17, 0);  // as do 16 to 17 of the next hidden units' instructions
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = next[e];
        }
        float l0 = 0.0f, l1 = 0.0f, l2 = 0.0f, l3 = 0.0f;
#pragma unroll 1
        for (int j = 0; j < 4; ++j) {
            float p[16];
#pragma unroll
            for (int i = 12; i >= 0; i -= 4) {
                const float4 b = *(const float4 *)(b2 + 32 * j + acc_row(half, i));
                const float4 w = *(const float4 *)(w3 + 32 * j + acc_row(half, i));
                const float bw[4] = {b.x, b.y, b.z, b.w}, ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = gelu(acc[0][i + e] + bw[e]);
                    p[i + e] = i >= 8 ? ww[e] * g : fmaf(ww[e], g, p[i + e + 8]);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                p[i] += p[i + 4];
                p[i] += __shfl_xor(p[i], 32, 64);
            }
            l0 = l1;
            l1 = l2;
            l2 = l3;
            l3 = (p[0] + p[2]) + (p[1] + p[3]);
            acc[0] = acc[1];
            acc[1] = acc[2];
            acc[2] = acc[3];
        }
        if (half == 0 && s < N) logits[s] = b3 + ((l0 + l1) + (l2 + l3));
    }
}

// the gradient is the sum of the blocks' contributions, in block order (deterministic);
// the loads of sixteen blocks are in flight at once
__device__ __forceinline__ float grad_sum(const float *__restrict__ partial, int slices, int64_t total, int64_t p) {
    float g = 0.0f;
    int j = 0;
    for (; j + 16 <= slices; j += 16) {
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = partial[(int64_t)(j + e) * total + p];
#pragma unroll
        for (int e = 0; e < 16; ++e) g += v[e];
    }
    for (; j < slices; ++j) g += partial[(int64_t)j * total + p];
    return g;
}

__global__ void grads_reduce_kernel(const float *__restrict__ partial, int slices, int64_t total,
                                    float *__restrict__ grad) {
    const int64_t p = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (p < total) grad[p] = grad_sum(partial, slices, total, p);
}

// Adam (Kingma and Ba, 2015) on fp32 master weights; refreshes the bf16 copy.
// The gradient is g[n] (slices = 0) or, in the training loop, the sum of the
// blocks' contributions, which then takes no kernel of its own (8.5 + 4.8 us for
// 32 blocks, now 4.7).
__global__ void adam_kernel(float *__restrict__ master, uint16_t *__restrict__ P,
                            float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ g, int slices, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= n) return;
    const float m0 = m[i], v0 = v[i], w0 = master[i];
    const float gi = slices ? grad_sum(g, slices, n, i) : g[i];
    const float mi = fmaf(1.0f - b1, gi, b1 * m0);
    const float vi = fmaf((1.0f - b2) * gi, gi, b2 * v0);
    m[i] = mi;
    v[i] = vi;
    const float w = w0 - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    master[i] = w;
    P[i] = f32_to_bf16(w);
}

// ---------------------------------------------------------------- features

// The front normalised per objective between its nadir (min) and ideal (max)
// (range 0 maps to 1).  Every block finds the range by itself, reading the
// front as a flat array with a multiple of m threads, so that a thread stays with
// one objective: 2048 points of four objectives 7.8 us for the range in one block
// and 4.2 for the division in a second launch, now 4.8 in one.
constexpr int kNormThreads = 1024, kNormBlocks = 256;

__global__ __launch_bounds__(kNormThreads) void front_norm_kernel(const int64_t *__restrict__ front, int64_t Pn, int m,
                                                                  float *__restrict__ yh) {
    __shared__ long long lo_sh[8], hi_sh[8];
    if (threadIdx.x < 8) {
        lo_sh[threadIdx.x] = INT64_MAX;
        hi_sh[threadIdx.x] = INT64_MIN;
    }
    __syncthreads();
    const int threads = kNormThreads / m * m, t = (int)threadIdx.x;
    const int64_t all = Pn * m;
    if (t < threads) {
        int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll 8
        for (int64_t i = t; i < all; i += threads) {
            const int64_t v = front[i];
            lo = v < lo ? v : lo;
            hi = v > hi ? v : hi;
        }
        atomicMin(&lo_sh[t % m], (long long)lo);
        atomicMax(&hi_sh[t % m], (long long)hi);
    }
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * kNormThreads + t; i < all; i += (int64_t)gridDim.x * kNormThreads) {
        const int k = (int)(i % m);
        const int64_t lo = lo_sh[k], hi = hi_sh[k];
        const double r = (double)hi - (double)lo;
        yh[i] = r > 0.0 ? (float)(((double)front[i] - (double)lo) / r) : 1.0f;
    }
}

// per front point: distance to the nearest other point and the fraction of
// points within 0.05 (itself included).  A block takes 64 points j, one per
// lane, and each of its sixteen waves a sixteenth of the points i, read at
// uniform addresses (scalar loads).  Squared distances are compared: the square
// root is monotone and correctly rounded, so sqrt(min d2) = min sqrt(d2), and
// sqrt(d2) <= 0.05f exactly when d2 <= kNear2, the largest float whose root is.
// Bound by the latency of the sixteenth's chain; 2048 points of four
// objectives: 866 us with a thread per j (8 blocks) and a root per pair, now 16.
constexpr float kNear2 = 0x1.47ae16p-9f;
constexpr int kLWaves = 16;

template <int M>
__global__ __launch_bounds__(64 * kLWaves) void front_local_kernel(const float *__restrict__ yh, int64_t Pn,
                                                                   float *__restrict__ nn, float *__restrict__ frac) {
    __shared__ float best_sh[kLWaves][64];
    __shared__ int32_t close_sh[kLWaves][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j0 = (int64_t)blockIdx.x * 64, j = j0 + lane;
    const bool active = j < Pn;
    float me[M];
#pragma unroll
    for (int k = 0; k < M; ++k) me[k] = active ? yh[j * M + k] : 0.0f;
    float best = INFINITY;
    int32_t close = 0;
    const int64_t per = (Pn + kLWaves - 1) / kLWaves;
    const int64_t i0 = min(Pn, wave * per), i1 = min(Pn, i0 + per);
    auto visit = [&](int64_t i, bool other) __attribute__((always_inline)) {
        float d2 = 0.0f;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const float d = yh[i * M + k] - me[k];
            d2 = fmaf(d, d, d2);
        }
        close += d2 <= kNear2 ? 1 : 0;
        best = fminf(best, other ? d2 : INFINITY);
    };
    // the block's own points need the test for the point itself
    const int64_t a = min(i1, max(i0, j0)), b = min(i1, max(i0, j0 + 64));
#pragma unroll 4
    for (int64_t i = i0; i < a; ++i) visit(i, true);
    for (int64_t i = a; i < b; ++i) visit(i, i != j);
#pragma unroll 4
    for (int64_t i = b; i < i1; ++i) visit(i, true);
    best_sh[wave][lane] = best;
    close_sh[wave][lane] = close;
    __syncthreads();
    if (wave != 0 || !active) return;
    int64_t n = 0;
    for (int w = 0; w < kLWaves; ++w) {
        best = fminf(best, best_sh[w][lane]);
        n += close_sh[w][lane];
    }
    nn[j] = Pn > 1 ? sqrtf(best) : 0.0f;
    frac[j] = (float)n / (float)Pn;
}

template <int M>
__device__ float angle(const float (&a)[M], const float *b) {
    // 2 atan2(|a^ - b^|, |a^ + b^|): accurate for nearly parallel vectors
    float na = 0.0f, nb = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        na = fmaf(a[k], a[k], na);
        nb = fmaf(b[k], b[k], nb);
    }
    na = sqrtf(na);
    nb = sqrtf(nb);
    float dm = 0.0f, dp = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const float u = a[k] / na, v = b[k] / nb;
        dm = fmaf(u - v, u - v, dm);
        dp = fmaf(u + v, u + v, dp);
    }
    return 2.0f * atan2f(sqrtf(dm), sqrtf(dp));
}

// A block takes 64 candidate weight vectors, one per lane; the front and the
// last round's hit and miss vectors are staged through LDS in chunks, and each
// of the four waves walks a quarter of every chunk, so that 65 536 candidates
// put four waves on every SIMD.  The waves' results are merged at the end.  The
// smallest angle to a set is taken at the set member with the largest cosine
// (the angle decreases with the cosine) and then evaluated accurately once.
// Ties go to the smallest index throughout, as in one pass over the set.  ALU
// bound: M + 12 instructions per front point (M products, eight for the sorted
// list of the largest values: with top[i-1] >= top[i], inserting v makes
// top[i] the median of the three; two for the
// maximiser, one against NaN).  65 536 candidates,
// 2048 points: 367 us with a thread per candidate and an insertion loop, now 88.
constexpr int kFChunk = 1024;
constexpr int kFWaves = kB / 64;

// this wave's quarter [i0, i1) of a chunk of cnt members
__device__ __forceinline__ void quarter(int cnt, int wave, int &i0, int &i1) {
    const int per = (cnt + kFWaves - 1) / kFWaves;
    i0 = min(cnt, wave * per);
    i1 = min(cnt, i0 + per);
}

template <int M>
__device__ __forceinline__ void best_cosine(const float (&u)[M], const float *__restrict__ vecs, int64_t count,
                                            float *stage, int wave, float &bc, int64_t &best) {
    bc = -INFINITY;
    best = -1;
    for (int64_t base = 0; base < count; base += kFChunk) {
        const int cnt = (int)(count - base < kFChunk ? count - base : kFChunk);
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += kB) {
            float nb = 0.0f;
#pragma unroll
            for (int k = 0; k < M; ++k) nb = fmaf(vecs[(base + i) * M + k], vecs[(base + i) * M + k], nb);
            const float inv = nb > 0.0f ? 1.0f / sqrtf(nb) : 0.0f;
#pragma unroll
            for (int k = 0; k < M; ++k) stage[i * M + k] = vecs[(base + i) * M + k] * inv;
        }
        __syncthreads();
        int i0, i1;
        quarter(cnt, wave, i0, i1);
        int at = -1;
#pragma unroll 4
        for (int i = i0; i < i1; ++i) {
            float d = 0.0f;
#pragma unroll
            for (int k = 0; k < M; ++k) d = fmaf(u[k], stage[i * M + k], d);
            at = d > bc ? i : at;
            bc = d > bc ? d : bc;
        }
        if (at >= 0) best = base + at;
    }
}

template <int M>
__global__ __launch_bounds__(kB) void features_kernel(const float *__restrict__ yh, int64_t Pn,
                                                      const float *__restrict__ nn, const float *__restrict__ frac,
                                                      const float *__restrict__ cands, int64_t N,
                                                      const float *__restrict__ hits, int64_t Hn,
                                                      const float *__restrict__ misses, int64_t Mn,
                                                      float *__restrict__ feat) {
    __shared__ __attribute__((aligned(16))) float stage[kFChunk * M];
    __shared__ float top_sh[kFWaves][8][64], cos_sh[kFWaves][2][64];
    __shared__ int64_t at_sh[kFWaves][3][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const bool active = c < N;
    float w[M], u[M];
    float nw = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        w[k] = active ? cands[c * M + k] : 0.0f;
        nw = fmaf(w[k], w[k], nw);
    }
    const float inv = nw > 0.0f ? 1.0f / sqrtf(nw) : 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) u[k] = w[k] * inv;
    // max, second and eighth largest of v_j = c . yh_j over the front, and the maximiser
    float top[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) top[i] = -INFINITY;
    int64_t jstar = 0;
    // (a product that is no number, from weights that are none, is left out)
    auto insert = [&](float v) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 7; i > 0; --i) top[i] = __builtin_amdgcn_fmed3f(top[i - 1], v, top[i]);
        top[0] = fmaxf(top[0], v);
    };
    for (int64_t base = 0; base < Pn; base += kFChunk) {
        const int cnt = (int)(Pn - base < kFChunk ? Pn - base : kFChunk);
        __syncthreads();
        for (int i = threadIdx.x; i < cnt * M; i += kB) stage[i] = yh[base * M + i];
        __syncthreads();
        int i0, i1;
        quarter(cnt, wave, i0, i1);
        int at = -1;
#pragma unroll 4
        for (int jj = i0; jj < i1; ++jj) {
            float v = 0.0f;
#pragma unroll
            for (int k = 0; k < M; ++k) v = fmaf(w[k], stage[jj * M + k], v);
            at = v > top[0] ? jj : at;  // first index on ties
            insert(fmaxf(v, -INFINITY));
        }
        if (at >= 0) jstar = base + at;
    }
    float hc, mc;
    int64_t bh, bm;
    best_cosine<M>(u, hits, Hn, stage, wave, hc, bh);
    best_cosine<M>(u, misses, Mn, stage, wave, mc, bm);
#pragma unroll
    for (int i = 0; i < 8; ++i) top_sh[wave][i][lane] = top[i];
    cos_sh[wave][0][lane] = hc;
    cos_sh[wave][1][lane] = mc;
    at_sh[wave][0][lane] = jstar;
    at_sh[wave][1][lane] = bh;
    at_sh[wave][2][lane] = bm;
    __syncthreads();
    if (wave != 0 || !active) return;
    // a wave's larger value, or its equal value at a smaller index, replaces the best so far
    auto better = [](float v, int64_t at, float &best, int64_t &best_at) {
        if (at >= 0 && (best_at < 0 || v > best || (v == best && at < best_at))) {
            best = v;
            best_at = at;
        }
    };
    for (int o = 1; o < kFWaves; ++o) {
        float t0 = top[0];
        if (top_sh[o][0][lane] > -INFINITY) better(top_sh[o][0][lane], at_sh[o][0][lane], t0, jstar);
#pragma unroll
        for (int i = 0; i < 8; ++i) insert(top_sh[o][i][lane]);
        better(cos_sh[o][0][lane], at_sh[o][1][lane], hc, bh);
        better(cos_sh[o][1][lane], at_sh[o][2][lane], mc, bm);
    }
    float f[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (Pn > 0) {
        f[0] = top[0];
        f[1] = Pn > 1 ? top[0] - top[1] : 0.0f;
        float last = top[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) last = i < Pn ? top[i] : last;
        f[2] = top[0] - last;
        f[3] = nn[jstar];
        f[4] = frac[jstar];
    }
    f[5] = bh >= 0 ? angle<M>(w, hits + bh * M) : 1.57079632679489662f;
    f[6] = bm >= 0 ? angle<M>(w, misses + bm * M) : 1.57079632679489662f;
    float dev = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) dev = fmaxf(dev, fabsf(w[k] - 1.0f / (float)M));
    f[7] = dev;
    // one MLP input row: the candidate followed by its eight features
    float *row = feat + c * (M + 8);
#pragma unroll
    for (int k = 0; k < M; ++k) row[k] = w[k];
#pragma unroll
    for (int i = 0; i < 8; ++i) row[M + i] = f[i];
}

// ---------------------------------------------------------------- selection and labels

// Gumbel-perturbed keys: the top k of score / tau + G (G standard Gumbel from
// the counter stream) is a sample of k items without replacement with
// probabilities proportional to exp(score / tau).
__device__ __forceinline__ float gumbel_key(float score, float inv_tau, uint64_t seed, int64_t i) {
    uint64_t z = seed + ((uint64_t)i + 1ull) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    const float u = ((float)(uint32_t)(z >> 40) + 0.5f) * 0x1p-24f;  // (0, 1)
    return score * inv_tau - logf(-logf(u));
}

// The key as an unsigned number in the order of the scores (the IEEE bit
// pattern made monotone; -0 is taken as +0).
__device__ __forceinline__ uint32_t key_bits(float f) {
    const uint32_t b = f == 0.0f ? 0u : __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// The key bits alone, for the ranks over all items.
__global__ void topk_bits_kernel(const float *__restrict__ s, int64_t N, bool gumbel, float inv_tau, uint64_t seed,
                                 uint32_t *__restrict__ key) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < N) key[i] = key_bits(gumbel ? gumbel_key(s[i], inv_tau, seed, i) : s[i]);
}

// comp[i] = (key bits, ~i): distinct, and larger is earlier in the result.
// Also clears `words` words that the following launches count in.
__global__ void topk_comp_kernel(const float *__restrict__ s, int64_t N, bool gumbel, float inv_tau, uint64_t seed,
                                 uint64_t *__restrict__ comp, uint32_t *__restrict__ clear, int words) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (blockIdx.x == 0)
        for (int w = threadIdx.x; w < words; w += kB) clear[w] = 0u;
    if (i >= N) return;
    const float f = gumbel ? gumbel_key(s[i], inv_tau, seed, i) : s[i];
    comp[i] = ((uint64_t)key_bits(f) << 32) | (uint32_t)~(uint32_t)i;
}

// One block's 64 items of a list (block b: items 64 b ..), one per lane, ranked
// against the n items of the list, a sixteenth per wave at uniform addresses:
// out[rank] = item for rank < k.  Two instructions per pair.
constexpr int kRankWaves = 16;
__device__ __forceinline__ void rank_block(const uint64_t *__restrict__ comp, int64_t n, int64_t k, int64_t b,
                                           int64_t *__restrict__ out, int32_t *sh) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = b * 64 + lane;
    const uint64_t mine = i < n ? comp[i] : 0ull;
    const int64_t per = ((n + kRankWaves - 1) / kRankWaves + 7) & ~int64_t(7);
    const int64_t j0 = min(n, wave * per), j1 = min(n, j0 + per);
    int32_t r = 0;
#pragma unroll 8
    for (int64_t j = j0; j < j1; ++j) r += comp[j] > mine ? 1 : 0;
    sh[wave * 64 + lane] = r;
    __syncthreads();
    if (wave != 0 || i >= n) return;
    int64_t rank = 0;
    for (int w = 0; w < kRankWaves; ++w) rank += sh[w * 64 + lane];
    if (rank < k) out[rank] = (int64_t)(uint32_t)~(uint32_t)mine;
}

// Every item's rank among n <= kRankAll, on the 32-bit keys in index order.  A
// block stages all keys in LDS and ranks 32 items; its 32 half-waves take a
// slice of the keys each, four per LDS read (the same address for the half).
// Equal keys rank by index: items before the block's own count when >=, items
// after it when >.
constexpr int kRankItems = 32;
constexpr int64_t kRankAll = 12288;  // 48 KB of keys
__global__ __launch_bounds__(64 * kRankWaves) void topk_rank_kernel(const uint32_t *__restrict__ key, int n, int64_t k,
                                                                    int64_t *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) uint32_t keys[];  // n rounded up to 4, zero padded
    __shared__ int32_t sh[2 * kRankWaves][kRankItems];
    const int n4 = (n + 3) & ~3;
#pragma unroll 4
    for (int j = 4 * threadIdx.x; j < n4; j += 4 * 64 * kRankWaves) {
        uint4 q = *(const uint4 *)(key + j);  // (the key buffer has room for a multiple of 4)
        q.y = j + 1 < n ? q.y : 0u;
        q.z = j + 2 < n ? q.z : 0u;
        q.w = j + 3 < n ? q.w : 0u;
        *(uint4 *)(keys + j) = q;
    }
    __syncthreads();
    const int item = threadIdx.x & (kRankItems - 1), slice = threadIdx.x / kRankItems;
    const int b0 = (int)blockIdx.x * kRankItems, i = b0 + item;
    const uint32_t mine = i < n ? keys[i] : 0u;
    const int per = ((n4 + 2 * kRankWaves - 1) / (2 * kRankWaves) + 3) & ~3;
    const int j0 = min(n4, slice * per), j1 = min(n4, j0 + per);
    const int a = min(j1, max(j0, b0)), b = min(j1, max(j0, b0 + kRankItems));  // all multiples of 4
    int32_t r = 0;
#pragma unroll 4
    for (int j = j0; j < a; j += 4) {
        const uint4 q = *(const uint4 *)(keys + j);
        r += (q.x >= mine) + (q.y >= mine) + (q.z >= mine) + (q.w >= mine);
    }
    for (int j = a; j < b; ++j) r += keys[j] > mine || (keys[j] == mine && j < i) ? 1 : 0;
#pragma unroll 4
    for (int j = b; j < j1; j += 4) {
        const uint4 q = *(const uint4 *)(keys + j);
        r += (q.x > mine) + (q.y > mine) + (q.z > mine) + (q.w > mine);
    }
    sh[slice][item] = r;
    __syncthreads();
    if (threadIdx.x >= kRankItems || i >= n) return;
    int64_t rank = 0;
#pragma unroll
    for (int w = 0; w < 2 * kRankWaves; ++w) rank += sh[w][item];
    if (rank < k) out[rank] = i;
}

// Selection for few of many: the key bits of the k-th item are found by three
// histograms (11, 11 and 10 bits), the items above it (fewer than k) are listed
// and ranked, and of the items equal to it the first by index fill the rest.
constexpr int kSelBins = 2048;
struct SelState {
    uint32_t bin[3], above[3];  // per level: the k-th item's bin, and the items in higher bins
    uint32_t listed;            // items appended to the list
    uint32_t pad;
};
constexpr int kSelMaxK = 4096;    // longest list to rank by pairs
constexpr int kSelChunks = 1024;  // blocks of the passes over the items (at most)

// Block-wide (256 threads): the bin of the k-th largest item (k >= 1, at most
// the items counted) and how many are in higher bins.
__device__ __forceinline__ void find_bin(const uint32_t *__restrict__ hist, uint32_t k, uint32_t &bin, uint32_t &above,
                                         uint32_t *sh) {
    constexpr int PER = kSelBins / kB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t c[PER], sum = 0;  // this thread's bins, from the top: kSelBins - 1 - (PER t + q)
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = hist[kSelBins - 1 - (PER * (int)threadIdx.x + q)];
        sum += c[q];
    }
    uint32_t s = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(s, off);
        if (lane >= off) s += o;
    }
    if (lane == 63) sh[wave] = s;
    __syncthreads();
    uint32_t before = s - sum;
    for (int w = 0; w < wave; ++w) before += sh[w];
    if (before < k && k <= before + sum) {
        uint32_t run = before;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (run < k && k <= run + c[q]) {
                sh[4] = kSelBins - 1 - (PER * threadIdx.x + q);
                sh[5] = run;
            }
            run += c[q];
        }
    }
    __syncthreads();
    bin = sh[4];
    above = sh[5];
    __syncthreads();
}

template <int LEVEL>
__global__ __launch_bounds__(kB) void topk_hist_kernel(const uint64_t *__restrict__ comp, int64_t N, int64_t chunk,
                                                       uint32_t k, uint32_t *__restrict__ hist, SelState *st) {
    __shared__ uint32_t h[kSelBins];
    __shared__ uint32_t sh[8];
    uint32_t prefix = 0;
    if constexpr (LEVEL > 0) {
        uint32_t bin, above;
        find_bin(hist + (LEVEL - 1) * kSelBins, LEVEL == 1 ? k : k - st->above[0], bin, above, sh);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->bin[LEVEL - 1] = bin;
            st->above[LEVEL - 1] = above;
        }
        prefix = LEVEL == 1 ? bin : (st->bin[0] << 11) | bin;
    }
    for (int i = threadIdx.x; i < kSelBins; i += kB) h[i] = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = min(N, i0 + chunk);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kB) {
        const uint32_t u = (uint32_t)(comp[i] >> 32);
        if (LEVEL == 0) atomicAdd(&h[u >> 21], 1u);
        if (LEVEL == 1 && (u >> 21) == prefix) atomicAdd(&h[(u >> 10) & 2047u], 1u);
        if (LEVEL == 2 && (u >> 10) == prefix) atomicAdd(&h[u & 1023u], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kB)
        if (h[i]) atomicAdd(&hist[LEVEL * kSelBins + i], h[i]);
}

// list[0 ..) = the items above the k-th key; equal[block] = the block's items at it.
__global__ __launch_bounds__(kB) void topk_collect_kernel(const uint64_t *__restrict__ comp, int64_t N, int64_t chunk,
                                                          uint32_t k, const uint32_t *__restrict__ hist, SelState *st,
                                                          uint64_t *__restrict__ list, uint32_t *__restrict__ equal) {
    __shared__ uint32_t sh[8];
    __shared__ uint32_t eq;
    if (threadIdx.x == 0) eq = 0u;
    uint32_t bin, above;
    find_bin(hist + 2 * kSelBins, k - st->above[0] - st->above[1], bin, above, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->bin[2] = bin;
        st->above[2] = above;
    }
    const uint32_t key = (st->bin[0] << 21) | (st->bin[1] << 10) | bin;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = min(N, i0 + chunk);
    for (int64_t c0 = i0; c0 < i1; c0 += 4 * kB) {  // one global atomic per 1024 items
        uint64_t c[4];
        uint32_t at[4];
        if (threadIdx.x == 0) sh[6] = 0u;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = c0 + r * kB + threadIdx.x;
            c[r] = i < i1 ? comp[i] : 0ull;
            const uint32_t u = (uint32_t)(c[r] >> 32);
            at[r] = i < i1 && u > key ? atomicAdd(&sh[6], 1u) : ~0u;
            if (i < i1 && u == key) atomicAdd(&eq, 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) sh[7] = sh[6] ? atomicAdd(&st->listed, sh[6]) : 0u;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (at[r] != ~0u) list[sh[7] + at[r]] = c[r];
    }
    __syncthreads();
    if (threadIdx.x == 0) equal[blockIdx.x] = eq;
}

// Blocks [0, rank_blocks): the listed items in order.  The others, one per
// chunk: the chunk's items at the k-th key, in index order, after them.
__global__ __launch_bounds__(64 * kRankWaves) void topk_emit_kernel(const uint64_t *__restrict__ comp, int64_t N,
                                                                    int64_t chunk, int64_t k, int rank_blocks,
                                                                    const SelState *__restrict__ st,
                                                                    const uint64_t *__restrict__ list,
                                                                    const uint32_t *__restrict__ equal,
                                                                    int64_t *__restrict__ out) {
    __shared__ int32_t sh[kRankWaves * 64];
    const int64_t above = (int64_t)st->above[0] + st->above[1] + st->above[2];
    if ((int)blockIdx.x < rank_blocks) {
        if ((int64_t)blockIdx.x * 64 < above) rank_block(list, above, k, blockIdx.x, out, sh);
        return;
    }
    const int b = (int)blockIdx.x - rank_blocks, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (equal[b] == 0) return;
    auto total = [&](int v) {
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) sh[wave] = v;
        __syncthreads();
        int s = 0;
        for (int w = 0; w < kRankWaves; ++w) s += sh[w];
        __syncthreads();
        return s;
    };
    const int before = total((int)threadIdx.x < b ? (int)equal[threadIdx.x] : 0);  // at most 1024 chunks
    const uint32_t key = (st->bin[0] << 21) | (st->bin[1] << 10) | st->bin[2];
    int64_t at = above + before;
    const int64_t i0 = (int64_t)b * chunk, i1 = min(N, i0 + chunk);
    for (int64_t i = i0 + threadIdx.x; i - (int64_t)threadIdx.x < i1 && at < k; i += 64 * kRankWaves) {
        const bool mine = i < i1 && (uint32_t)(comp[i] >> 32) == key;
        const uint64_t mask = __ballot(mine);
        if (lane == 0) sh[wave] = __popcll(mask);
        __syncthreads();
        int pre = 0, all = 0;
        for (int w = 0; w < kRankWaves; ++w) {
            if (w < wave) pre += sh[w];
            all += sh[w];
        }
        const int64_t pos = at + pre + __popcll(mask & ((1ull << lane) - 1ull));
        if (mine && pos < k) out[pos] = i;
        at += all;
        __syncthreads();
    }
}

// The radix sort's keys: ascending unsigned order is descending score order.
// Block 0 also stores the item and digit pass counts that the sort reads from
// device memory.
__global__ void topk_key_kernel(const float *__restrict__ s, int64_t N, bool gumbel, float inv_tau, uint64_t seed,
                                uint64_t *__restrict__ key, int32_t *__restrict__ val, int64_t *__restrict__ d_n,
                                int32_t *__restrict__ d_passes) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i == 0) {
        *d_n = N;
        *d_passes = 4;
    }
    if (i >= N) return;
    const float f = gumbel ? gumbel_key(s[i], inv_tau, seed, i) : s[i];
    key[i] = (uint64_t)(uint32_t)~key_bits(f);
    val[i] = (int32_t)i;
}

__global__ void topk_out_kernel(const int32_t *__restrict__ val, int64_t k, int64_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < k) out[i] = val[i];
}

__global__ void labels_kernel(const int64_t *__restrict__ keep, const int64_t *__restrict__ num_keep,
                              int64_t archive, int R, int64_t W, float *__restrict__ labels) {
    const int64_t K = *num_keep;
    for (int64_t t = (int64_t)blockIdx.x * kB + threadIdx.x; t < K; t += (int64_t)gridDim.x * kB) {
        const int64_t s = keep[t];
        if (s >= archive) {
            const int64_t w = (s - archive) / R;
            if (w < W) labels[w] = 1.0f;
        }
    }
}

__global__ void zero_f32_kernel(float *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

__global__ void gather_rows_kernel(const uint32_t *__restrict__ src, int width,
                                   const int64_t *__restrict__ idx, const int64_t *__restrict__ count,
                                   int64_t cap, uint32_t *__restrict__ dst) {
    const int64_t K = *count < cap ? *count : cap;
    for (int64_t t = (int64_t)blockIdx.x * kB + threadIdx.x; t < K * width; t += (int64_t)gridDim.x * kB) {
        const int64_t r = t / width, c = t % width;
        dst[t] = src[idx[r] * width + c];
    }
}

unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + kB - 1) / kB); }

}  // namespace

int64_t mlp_param_count(int D) { return offsets(D).total; }

static int64_t grad_blocks(int64_t B) { return (B + kS - 1) / kS; }

size_t mlp_backward_ws_bytes(int D, int64_t B) {
    return align256(sizeof(float) * (size_t)std::max<int64_t>(grad_blocks(B), 1) *
                    (size_t)offsets(std::max(D, 1)).total);
}

size_t mlp_forward_ws_bytes(int64_t N) {
    (void)N;
    return 256;  // the fused forward keeps everything on chip
}

// A wave alone with a tile needs 30 us however few there are, a block with a tile
// 11, one per CU at a time: 8192 samples 11 against 30 us, 16 384 19 / 30, 24 000
// 27.5 / 30, and a fourth round of the blocks would be slower than the 30 us of 32 768.
constexpr int64_t kRowsMin = 24576;
// Four blocks per tile while they all run at once, one per CU: 64 tiles 15.6 us
// split, 23 whole; at 65 tiles the split would take a second round.
constexpr int64_t kSplitMax = 64;

void launch_mlp_forward(const uint16_t *P, int D, const float *X, int64_t N, float *logits, void *ws,
                        hipStream_t st) {
    (void)ws;
    QAIA_CHECK(D >= 1 && D <= kMaxD, QAIA_INVALID_ARGUMENT, "input width must be in [1, 16]");
    if (N == 0) return;
    const int64_t blocks = grad_blocks(N);
    QAIA_CHECK(blocks <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many samples");
    if (N > kRowsMin) {
        // 256 blocks give up to eight tiles per CU to different SIMDs; above, two blocks share a CU
        // (262 144 samples 168 us with 256 blocks, 158 with 512; 16 385 29 and 43)
        const unsigned rows_blocks = blocks <= 256 * kRWaves ? 256 : 512;
        const auto k = D <= 4    ? mlp_rows_kernel<1>
                       : D <= 8  ? mlp_rows_kernel<2>
                       : D <= 12 ? mlp_rows_kernel<3>
                                 : mlp_rows_kernel<4>;
        hipLaunchKernelGGL(k, dim3((unsigned)rows_blocks), dim3(64 * kRWaves), 0, st, P, D, X, N,
                           logits);
    } else {
        hipLaunchKernelGGL((mlp_tile_kernel<false, 1>), dim3((unsigned)blocks), dim3(kT), 0, st, P, D, X, N,
                           (const float *)nullptr, logits, (float *)nullptr);
    }
    QAIA_HIP(hipGetLastError());
}

static int launch_mlp_partial(const uint16_t *P, int D, const float *X, const float *y, int64_t B, float *logits,
                              float *partial, hipStream_t st) {
    QAIA_CHECK(D >= 1 && D <= kMaxD, QAIA_INVALID_ARGUMENT, "input width must be in [1, 16]");
    QAIA_CHECK(B >= 1, QAIA_INVALID_ARGUMENT, "batch must be >= 1");
    const int64_t blocks = grad_blocks(B);
    QAIA_CHECK(blocks <= 65535, QAIA_INVALID_ARGUMENT, "batch too large");
    if (blocks <= kSplitMax)
        hipLaunchKernelGGL((mlp_tile_kernel<true, 4>), dim3((unsigned)blocks, 4), dim3(kT), 0, st, P, D, X, B, y,
                           logits, partial);
    else
        hipLaunchKernelGGL((mlp_tile_kernel<true, 1>), dim3((unsigned)blocks), dim3(kT), 0, st, P, D, X, B, y, logits,
                           partial);
    QAIA_HIP(hipGetLastError());
    return (int)blocks;
}

void launch_mlp_backward(const uint16_t *P, int D, const float *X, const float *y, int64_t B,
                         float *grad, float *loss_logits, void *ws, hipStream_t st) {
    float *partial = (float *)ws;
    const int blocks = launch_mlp_partial(P, D, X, y, B, loss_logits, partial, st);
    const int64_t total = offsets(D).total;
    hipLaunchKernelGGL(grads_reduce_kernel, dim3(blocks_for(total)), dim3(kB), 0, st, partial, blocks, total, grad);
    QAIA_HIP(hipGetLastError());
}

static void launch_adam_step(float *master, uint16_t *P, float *m, float *v, const float *g, int slices, int64_t n,
                             int step, float lr, float b1, float b2, float eps, hipStream_t st) {
    QAIA_CHECK(step >= 1, QAIA_INVALID_ARGUMENT, "Adam step counts from 1");
    const float c1 = (float)(1.0 - std::pow((double)b1, step));
    const float c2 = (float)(1.0 - std::pow((double)b2, step));
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(kB), 0, st, master, P, m, v, g, slices, n, lr, b1,
                       b2, eps, c1, c2);
    QAIA_HIP(hipGetLastError());
}

void launch_adam(float *master, uint16_t *P, float *m, float *v, const float *g, int64_t n, int step,
                 float lr, float b1, float b2, float eps, hipStream_t st) {
    launch_adam_step(master, P, m, v, g, 0, n, step, lr, b1, b2, eps, st);
}

// ---------------------------------------------------------------- training loop

namespace {
__global__ void train_count_kernel(int64_t *c, int64_t n) {
    if (threadIdx.x == 0) *c = n;
}
}  // namespace

struct TrainLayout {
    size_t zeros, perm, xp, yp, count, bw, tk, total;
};

static TrainLayout train_layout(int D, int64_t n, int64_t B) {
    TrainLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += align256(bytes);
        return o;
    };
    const size_t nz = (size_t)std::max<int64_t>(n, 1);
    L.zeros = take(sizeof(float) * nz);
    L.perm = take(sizeof(int64_t) * nz);
    L.xp = take(sizeof(float) * nz * (size_t)D);
    L.yp = take(sizeof(float) * nz);
    L.count = take(sizeof(int64_t));
    L.bw = take(mlp_backward_ws_bytes(D, B));
    L.tk = take(topk_ws_bytes(n));
    L.total = off;
    return L;
}

size_t mlp_train_ws_bytes(int D, int64_t n, int64_t batch) {
    return train_layout(std::max(D, 1), std::max<int64_t>(n, 1), std::min(std::max<int64_t>(batch, 1), std::max<int64_t>(n, 1))).total;
}

// `steps` Adam steps on minibatches of min(batch, n) rows: minibatch t is
// window t mod (n / B) of a random permutation of the rows, drawn afresh at
// the start of every pass as the Gumbel top-k of n equal scores with seed
// `seed + 104729 * (first_step + t)`; the Adam step counter runs from
// first_step.
void launch_mlp_train(float *master, uint16_t *P, float *m1, float *m2, int D, const float *X, const float *y,
                      int64_t n, int64_t batch, int steps, int first_step, float lr, uint64_t seed, void *ws,
                      size_t ws_bytes, hipStream_t st) {
    QAIA_CHECK(D >= 1 && D <= kMaxD, QAIA_INVALID_ARGUMENT, "input width must be in [1, 16]");
    QAIA_CHECK(n >= 1 && batch >= 1 && steps >= 0 && first_step >= 1, QAIA_INVALID_ARGUMENT,
               "need n >= 1, batch >= 1, steps >= 0, first_step >= 1");
    const int64_t B = std::min(batch, n), per_pass = n / B;
    const TrainLayout L = train_layout(D, n, B);
    QAIA_CHECK(ws_bytes >= L.total, QAIA_WORKSPACE_TOO_SMALL, "training workspace too small");
    char *b = (char *)ws;
    float *zeros = (float *)(b + L.zeros), *xp = (float *)(b + L.xp), *yp = (float *)(b + L.yp);
    int64_t *perm = (int64_t *)(b + L.perm), *cnt = (int64_t *)(b + L.count);
    const int64_t total = offsets(D).total;
    hipLaunchKernelGGL(zero_f32_kernel, dim3(blocks_for(n)), dim3(kB), 0, st, zeros, n);
    hipLaunchKernelGGL(train_count_kernel, dim3(1), dim3(64), 0, st, cnt, n);
    QAIA_HIP(hipGetLastError());
    for (int t = 0; t < steps; ++t) {
        const int64_t win = t % per_pass;
        if (win == 0) {
            launch_topk(zeros, n, n, 1.0f, seed + 104729ull * (uint64_t)(first_step + t), perm, b + L.tk,
                        topk_ws_bytes(n), st);
            launch_gather_rows((const uint32_t *)X, D, perm, cnt, n, (uint32_t *)xp, st);
            launch_gather_rows((const uint32_t *)y, 1, perm, cnt, n, (uint32_t *)yp, st);
        }
        float *partial = (float *)(b + L.bw);
        const int blocks = launch_mlp_partial(P, D, xp + win * B * D, yp + win * B, B, nullptr, partial, st);
        launch_adam_step(master, P, m1, m2, partial, blocks, total, first_step + t, lr, 0.9f, 0.999f, 1e-8f, st);
    }
}

size_t features_ws_bytes(int64_t Pn, int m) {
    return align256(sizeof(float) * (size_t)std::max<int64_t>(Pn, 1) * m) +
           2 * align256(sizeof(float) * (size_t)std::max<int64_t>(Pn, 1));
}

void launch_features(const int64_t *front, int64_t Pn, int m, const float *cands, int64_t N,
                     const float *hits, int64_t Hn, const float *misses, int64_t Mn, float *feat,
                     void *ws, size_t ws_bytes, hipStream_t st) {
    QAIA_CHECK(m >= 1 && m <= 8, QAIA_INVALID_ARGUMENT, "m must be in [1, 8]");
    QAIA_CHECK(ws_bytes >= features_ws_bytes(Pn, m), QAIA_WORKSPACE_TOO_SMALL, "feature workspace too small");
    if (N == 0) return;
    char *b = (char *)ws;
    size_t off = 0;
    float *yh = (float *)(b + off);
    off += align256(sizeof(float) * (size_t)std::max<int64_t>(Pn, 1) * m);
    float *nn = (float *)(b + off);
    off += align256(sizeof(float) * (size_t)std::max<int64_t>(Pn, 1));
    float *frac = (float *)(b + off);
    if (Pn > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>((Pn * m + kNormThreads - 1) / kNormThreads, kNormBlocks);
        hipLaunchKernelGGL(front_norm_kernel, dim3(grid), dim3(kNormThreads), 0, st, front, Pn, m, yh);
    }
#define QAIA_FEATURES(MM)                                                                                     \
    case MM:                                                                                                  \
        if (Pn > 0)                                                                                           \
            hipLaunchKernelGGL(front_local_kernel<MM>, dim3((unsigned)((Pn + 63) / 64)), dim3(64 * kLWaves), 0, st, yh, \
                               Pn, nn, frac);                                                                 \
        hipLaunchKernelGGL(features_kernel<MM>, dim3((unsigned)((N + 63) / 64)), dim3(kB), 0, st, yh, Pn, nn, frac, cands, N, \
                           hits, Hn, misses, Mn, feat);                                                       \
        break;
    switch (m) {
        QAIA_FEATURES(1)
        QAIA_FEATURES(2)
        QAIA_FEATURES(3)
        QAIA_FEATURES(4)
        QAIA_FEATURES(5)
        QAIA_FEATURES(6)
        QAIA_FEATURES(7)
        QAIA_FEATURES(8)
        default: throw Error{QAIA_UNSUPPORTED, "features support 1..8 objectives"};
    }
#undef QAIA_FEATURES
    QAIA_HIP(hipGetLastError());
}

size_t topk_ws_bytes(int64_t N) {
    const size_t n = (size_t)std::max<int64_t>(N, 1);
    return 2 * align256(sizeof(uint64_t) * n) + 2 * align256(sizeof(int32_t) * n) + align256(4 * radix_hist_words(N)) +
           align256(4 * 256) + align256(64);
}

// Three ways to the same order, by size:
//  - up to kRankAll items: every item's rank by comparing all pairs, two
//    launches (8192 items, all returned: 17 us; the radix sort's fourteen
//    launches took 120 us at 8192 items and 134 at 65 536; past 12 288 items
//    the pairs take as long as the selection);
//  - more items, at most kSelMaxK returned: selection, six launches (65 536
//    items, 922 returned: 28 us);
//  - otherwise the stable radix sort.
void launch_topk(const float *scores, int64_t N, int64_t k, float temperature, uint64_t seed, int64_t *idx_out,
                 void *ws, size_t ws_bytes, hipStream_t st) {
    QAIA_CHECK(N >= 1 && N < (int64_t(1) << 31), QAIA_INVALID_ARGUMENT, "N must be in [1, 2^31)");
    QAIA_CHECK(k >= 0 && k <= N, QAIA_INVALID_ARGUMENT, "k must be in [0, N]");
    QAIA_CHECK(ws_bytes >= topk_ws_bytes(N), QAIA_WORKSPACE_TOO_SMALL, "top-k workspace too small");
    QAIA_CHECK(temperature >= 0.0f && std::isfinite(temperature), QAIA_INVALID_ARGUMENT,
               "temperature must be finite and >= 0");
    if (k == 0) return;
    char *b = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = b + off;
        off += align256(bytes);
        return p;
    };
    uint64_t *keyA = (uint64_t *)take(sizeof(uint64_t) * (size_t)N), *keyB = (uint64_t *)take(sizeof(uint64_t) * (size_t)N);
    int32_t *valA = (int32_t *)take(sizeof(int32_t) * (size_t)N), *valB = (int32_t *)take(sizeof(int32_t) * (size_t)N);
    uint32_t *hist = (uint32_t *)take(4 * radix_hist_words(N)), *total = (uint32_t *)take(4 * 256);
    char *small = take(64);
    const bool gumbel = temperature > 0.0f;
    const float inv_tau = gumbel ? 1.0f / temperature : 0.0f;
    const dim3 items(blocks_for(N)), block(kB), rank_block(64 * kRankWaves);
    if (N <= kRankAll) {
        uint32_t *bits = (uint32_t *)keyA;
        hipLaunchKernelGGL(topk_bits_kernel, items, block, 0, st, scores, N, gumbel, inv_tau, seed, bits);
        hipLaunchKernelGGL(topk_rank_kernel, dim3((unsigned)((N + kRankItems - 1) / kRankItems)), rank_block,
                           4 * (size_t)((N + 3) & ~int64_t(3)), st, bits, (int)N, k, idx_out);
        QAIA_HIP(hipGetLastError());
        return;
    }
    if (k <= kSelMaxK) {
        // in keyB's memory (8 N > 131 072 bytes): the list, the histograms, the state, the chunks' counts
        uint64_t *list = keyB;
        uint32_t *bins = (uint32_t *)(list + kSelMaxK);
        SelState *state = (SelState *)(bins + 3 * kSelBins);
        uint32_t *equal = (uint32_t *)(state + 1);
        static_assert(8 * kSelMaxK + 12 * kSelBins + sizeof(SelState) + 4 * kSelChunks <= 8 * (size_t)kRankAll, "fits");
        const int64_t chunk = ((N + kSelChunks - 1) / kSelChunks + 1023) / 1024 * 1024;
        const unsigned chunks = (unsigned)((N + chunk - 1) / chunk);
        const int rank_blocks = (int)((k + 63) / 64);
        hipLaunchKernelGGL(topk_comp_kernel, items, block, 0, st, scores, N, gumbel, inv_tau, seed, keyA, bins,
                           3 * kSelBins + (int)(sizeof(SelState) / 4));
        hipLaunchKernelGGL(topk_hist_kernel<0>, dim3(chunks), block, 0, st, keyA, N, chunk, (uint32_t)k, bins, state);
        hipLaunchKernelGGL(topk_hist_kernel<1>, dim3(chunks), block, 0, st, keyA, N, chunk, (uint32_t)k, bins, state);
        hipLaunchKernelGGL(topk_hist_kernel<2>, dim3(chunks), block, 0, st, keyA, N, chunk, (uint32_t)k, bins, state);
        hipLaunchKernelGGL(topk_collect_kernel, dim3(chunks), block, 0, st, keyA, N, chunk, (uint32_t)k, bins, state, list,
                           equal);
        hipLaunchKernelGGL(topk_emit_kernel, dim3(rank_blocks + chunks), rank_block, 0, st, keyA, N, chunk, k, rank_blocks,
                           state, list, equal, idx_out);
        QAIA_HIP(hipGetLastError());
        return;
    }
    int64_t *d_n = (int64_t *)small;
    int32_t *d_passes = (int32_t *)(small + 8);
    // stable: equal scores keep increasing index order; four passes leave the result in A
    hipLaunchKernelGGL(topk_key_kernel, items, block, 0, st, scores, N, gumbel, inv_tau, seed, keyA, valA, d_n, d_passes);
    QAIA_HIP(hipGetLastError());
    for (int pass = 0; pass < 4; ++pass) {
        const bool even = (pass & 1) == 0;
        radix_pass(even ? keyA : keyB, even ? valA : valB, even ? keyB : keyA, even ? valB : valA, N, d_n, d_passes,
                   pass, hist, total, st);
    }
    hipLaunchKernelGGL(topk_out_kernel, dim3(blocks_for(k)), dim3(kB), 0, st, valA, k, idx_out);
    QAIA_HIP(hipGetLastError());
}

void launch_labels(const int64_t *keep, const int64_t *num_keep, int64_t archive, int R, int64_t W,
                   float *labels, hipStream_t st) {
    QAIA_CHECK(R >= 1 && W >= 0 && archive >= 0, QAIA_INVALID_ARGUMENT, "bad label arguments");
    if (W == 0) return;
    hipLaunchKernelGGL(zero_f32_kernel, dim3(blocks_for(W)), dim3(kB), 0, st, labels, W);
    hipLaunchKernelGGL(labels_kernel, dim3(1024), dim3(kB), 0, st, keep, num_keep, archive, R, W, labels);
    QAIA_HIP(hipGetLastError());
}

void launch_gather_rows(const uint32_t *src, int width, const int64_t *idx, const int64_t *count,
                        int64_t cap, uint32_t *dst, hipStream_t st) {
    QAIA_CHECK(width >= 1 && cap >= 0, QAIA_INVALID_ARGUMENT, "bad gather arguments");
    hipLaunchKernelGGL(gather_rows_kernel, dim3(1024), dim3(kB), 0, st, src, width, idx, count, cap, dst);
    QAIA_HIP(hipGetLastError());
}

}  // namespace qaia
