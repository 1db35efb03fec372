// Dense SB for small graphs: the whole run in one launch.
//
// The staged step kernels (dense.hip) launch once per step, read and write x, y
// and Phi through HBM each time, pad n to a multiple of 128 and run the matrix
// product, the update and the noise one after the other.  Up to kResidentMaxN
// spins a block can instead keep 32 columns for all T steps: it has one wave per
// 32 spins, each holding the x and y of its 32 x 32 tile in registers in the
// MFMA accumulator layout, and Phi (all spins of the 32 columns) in LDS, double
// buffered, one barrier per step.  The J operands stream from L2 every step, each
// wave reading only its own 32 rows, from images in fragment order (one
// contiguous 1 KB per operand; 16 bytes per cycle and CU at the FP32 matrix
// rate).  Several waves per SIMD overlap one block's update and Gaussian draws
// with another's matrix product.  k-groups past n are skipped: their products are
// exact zeros.
//
// Every accumulator receives the k-groups in the staged kernels' order with the
// same lane mapping, and the update is the same sequence of operations, so the
// trajectories are theirs bit for bit.
//
// Bound by the FP32 matrix rate where columns fill the GPU (512 spins, m = 4, 8192
// columns: 117 us per step of 111 at the rate a large product reaches, 135 staged),
// with few columns by one block's chain of MFMAs (past 256 spins such calls take the
// thin tiles of dense.hip instead, its launch_dense says where).  Per step, staged -> here:
// n = 256, m = 3, 8192 columns 56 -> 26, BF16 15.0 -> 5.2, FP8 12.4 -> 3.5; n = 70,
// m = 4, 200 columns 40 -> 5.7 (the launches).  512 spins are sixteen waves; past
// that a wave would need two row tiles and their registers.
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "device_common.hpp"
#include "internal.hpp"

namespace qaia {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kB = 256;
constexpr int kCols = 32;  // columns per tile

// KG spins per k-group; a lane of half h holds spins KG h / 2 .. of it
template <int PREC> struct Op;
template <> struct Op<QAIA_FP32> { typedef f32x4 V; typedef float T; static constexpr int KG = 8; };
template <> struct Op<QAIA_BF16> { typedef bf16x8 V; typedef uint16_t T; static constexpr int KG = 16; };
template <> struct Op<QAIA_FP8> { typedef i32x8 V; typedef uint8_t T; static constexpr int KG = 64; };

template <int PREC>
__host__ __device__ constexpr int kgroups(int n) { return (n + Op<PREC>::KG - 1) / Op<PREC>::KG; }
// LDS bytes of one column's Phi: whole k-groups and 16 bytes, an odd number of
// 16-byte parts, so that the 32 columns' parts fall on distinct banks
template <int PREC>
__host__ __device__ constexpr int phi_pitch(int n) {
    const int b = kgroups<PREC>(n) * Op<PREC>::KG * (int)sizeof(typename Op<PREC>::T) + 16;
    return (b / 16) % 2 ? b : b + 16;
}

__device__ __forceinline__ int acc_row(int half, int i) { return (i >> 2) * 8 + half * 4 + (i & 3); }

template <int PREC>
__device__ __forceinline__ void mma(const typename Op<PREC>::V &a, const typename Op<PREC>::V &b, f16v &c) {
    if constexpr (PREC == QAIA_FP32) {
#pragma unroll
        for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], c, 0, 0, 0);
    } else if constexpr (PREC == QAIA_BF16) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    } else {
        c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
    }
}

// Images in fragment order: element j of lane (h, i) of fragment (k, r, g) is
// J[k][32 r + i][KG g + KG / 2 h + j].
template <int PREC>
__global__ __launch_bounds__(kB) void fragment_kernel(const typename Op<PREC>::T *__restrict__ J, int m, int Np, int n,
                                                      typename Op<PREC>::T *__restrict__ out) {
    constexpr int KG = Op<PREC>::KG, H = KG / 2;
    const int tiles = (n + 31) / 32, groups = kgroups<PREC>(n);
    const int64_t idx = (int64_t)blockIdx.x * kB + threadIdx.x, all = (int64_t)m * tiles * groups * 64 * H;
    if (idx >= all) return;
    const int j = (int)(idx % H), lane = (int)(idx / H % 64);
    const int64_t f = idx / H / 64;
    const int g = (int)(f % groups), r = (int)(f / groups % tiles), k = (int)(f / groups / tiles);
    out[idx] = J[((int64_t)k * Np + 32 * r + (lane & 31)) * Np + KG * g + H * (lane >> 5) + j];
}

struct ResidentArgs {
    const void *J;  // fragment-order image
    const float *weights;
    const double *c0s;
    const float *kt_tab;
    const float *jscale;  // [m] for this precision
    float dta0, dt_alpha, amp;
    double dt;
    int n, m, R, T, tiles;  // tiles: row tiles = waves per column tile
    int64_t cols;
    uint64_t seed, offset;
    uint64_t *spins;
    int words;
    float *trace;
    int trace_steps;
};

// this wave's 32 spins of each column, the halves' bits joined
__device__ __forceinline__ void read_out(const ResidentArgs &a, int r, int half, int lr, int64_t col, bool mine,
                                         const float *x) {
    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = r * 32 + acc_row(half, i);
        if (row < a.n && x[i] < 0.0f) bits |= 1u << acc_row(half, i);
    }
    bits |= (uint32_t)__shfl_xor((int)bits, 32);
    if (half == 0 && mine) {
        const bool valid = a.c0s[col / a.R] >= 0.0;
        uint32_t *out = (uint32_t *)(a.spins + col * a.words);
        out[r] = valid ? bits : 0u;
        if (r == a.tiles - 1 && a.tiles < 2 * a.words) out[r + 1] = 0u;  // the last 64-bit word's upper half
    }
}

template <int PREC, int M, bool DSB, bool NOISE, bool AHEAD>
__device__ __forceinline__ void resident_body(const ResidentArgs &a, char *lds) {
    typedef typename Op<PREC>::V V;
    typedef typename Op<PREC>::T T;
    constexpr int KG = Op<PREC>::KG;
    const int lane = threadIdx.x & 63, half = lane >> 5, lr = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = wave % a.tiles, ct = wave / a.tiles;  // row tile, column tile of the block
    const int per_block = (int)(blockDim.x >> 6) / a.tiles;
    const int64_t col = ((int64_t)blockIdx.x * per_block + ct) * kCols + lr;
    const bool mine = col < a.cols;
    const int groups = kgroups<PREC>(a.n), pitch = phi_pitch<PREC>(a.n);
    char *const phi0 = lds + (size_t)ct * 2 * kCols * pitch;  // this column tile's two buffers
    const uint64_t g = (uint64_t)col + a.offset;

    float cf[M];
    {
        const int64_t w = mine ? col / a.R : 0;
        const double c0 = mine ? a.c0s[w] : -1.0;
#pragma unroll
        for (int k = 0; k < M; ++k)
            cf[k] = c0 >= 0.0 ? (float)(-a.dt * c0 * (double)a.weights[w * M + k] * (double)a.jscale[k]) : 0.0f;
    }
    float x[16], y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = r * 32 + acc_row(half, i);
        const bool live = mine && row < a.n;
        x[i] = live ? init_value(a.seed, init_counter(g, a.n, row, 0), a.amp) : 0.0f;
        y[i] = live ? init_value(a.seed, init_counter(g, a.n, row, 1), a.amp) : 0.0f;
    }
    // this lane's Phi values, four consecutive spins at a time
    auto put_phi = [&](char *buf) __attribute__((always_inline)) {
        T *p = (T *)(buf + lr * pitch) + r * 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = acc_row(half, 4 * q);
            if (r * 32 + row >= groups * KG) continue;  // (both multiples of 4)
            const float *v = x + 4 * q;
            if constexpr (PREC == QAIA_FP32) {
                *(f32x4 *)(p + row) = DSB ? f32x4{sgn1(v[0]), sgn1(v[1]), sgn1(v[2]), sgn1(v[3])}
                                          : f32x4{v[0], v[1], v[2], v[3]};
            } else if constexpr (PREC == QAIA_BF16) {
                uint2 b;
                b.x = (v[0] >= 0.0f ? 0x3F80u : 0xBF80u) | ((v[1] >= 0.0f ? 0x3F80u : 0xBF80u) << 16);
                b.y = (v[2] >= 0.0f ? 0x3F80u : 0xBF80u) | ((v[3] >= 0.0f ? 0x3F80u : 0xBF80u) << 16);
                *(uint2 *)(p + row) = b;
            } else {
                uint32_t b = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) b |= (v[e] >= 0.0f ? 0x38u : 0xB8u) << (8 * e);
                *(uint32_t *)(p + row) = b;
            }
        }
    };
    // Phi past the last row tile (k-groups of 64 spins) stays zero
    for (int i = threadIdx.x * 4; i < per_block * 2 * kCols * pitch; i += blockDim.x * 4) *(uint32_t *)(lds + i) = 0u;
    __syncthreads();
    put_phi(phi0);
    __syncthreads();

    // Fragment (k, r, q) through a buffer descriptor: a scalar offset and one
    // register for the lane (with ordinary loads the compiler keeps M 64-bit
    // addresses per lane, which spilled at M = 4 and sixteen waves: 146 us per step,
    // now 120; the 2 to 19 registers that are still too few there are read back from
    // scratch once per step, not in the loop over the fragments).
    constexpr int FB = 64 * (int)sizeof(V);  // bytes of a fragment
    const int kstride = a.tiles * groups * FB;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.J, 0, M * kstride, 0x00027000);
    const int rbase = r * groups * FB, voff = lane * (int)sizeof(V);
    auto load_a = [&](int k, int q) __attribute__((always_inline)) {
        const int so = rbase + k * kstride + q * FB;
        if constexpr (sizeof(V) == 16) {
            return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, so, 0));
        } else {
            struct Two { u32x4 lo, hi; } two{__builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, so, 0),
                                             __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + 16, so, 0)};
            return __builtin_bit_cast(V, two);
        }
    };
    // the noise counter of this lane's first spin at step t: (g T + t) n + row
    constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;
    uint64_t zb = 0;
    if constexpr (NOISE)
        zb = (a.seed ^ kNoiseKey) + (g * (uint64_t)a.T * (uint64_t)a.n + (uint64_t)(r * 32 + 4 * half) + 1ull) * kGamma;
    const uint64_t zstep = (uint64_t)a.n * kGamma;

    for (int t = 0; t < a.T; ++t) {
        const float kt = a.kt_tab[t];
        const char *pc = phi0 + (t & 1) * kCols * pitch + lr * pitch + half * (KG / 2) * sizeof(T);
        f16v acc[M];
#pragma unroll
        for (int k = 0; k < M; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[k][i] = 0.0f;
        V av[M];
        if constexpr (!AHEAD) {  // sixteen waves: 128 registers leave no room for a second set, four waves a SIMD hide the loads
#pragma unroll 1
            for (int q = 0; q < groups; ++q) {
#pragma unroll
                for (int k = 0; k < M; ++k) av[k] = load_a(k, q);
                const V b = *(const V *)(pc + (size_t)q * KG * sizeof(T));
#pragma unroll
                for (int k = 0; k < M; ++k) mma<PREC>(av[k], b, acc[k]);
            }
        } else {
#pragma unroll
        for (int k = 0; k < M; ++k) {
            av[k] = load_a(k, 0);
            asm volatile("" : "+v"(av[k]));  // opaque: the compiler would sink the prefetch below to the point of use
        }
        for (int q = 0; q < groups; ++q) {
            V nx[M];
            const int qn = q + 1 < groups ? q + 1 : q;
#pragma unroll
            for (int k = 0; k < M; ++k) nx[k] = load_a(k, qn);
            const V b = *(const V *)(pc + (size_t)q * KG * sizeof(T));
#pragma unroll
            for (int k = 0; k < M; ++k) mma<PREC>(av[k], b, acc[k]);
#pragma unroll
            for (int k = 0; k < M; ++k) av[k] = nx[k];
        }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = r * 32 + acc_row(half, i);
            float h = 0.0f;
#pragma unroll
            for (int k = 0; k < M; ++k) h = fmaf(cf[k], acc[k][i], h);
            float yn = fmaf(kt, x[i], y[i]) + h;
            if constexpr (NOISE)
                if (mine && row < a.n)
                    yn = fmaf(a.dt_alpha, noise_from(zb + (uint64_t)((i >> 2) * 8 + (i & 3)) * kGamma), yn);
            float xn = fmaf(a.dta0, yn, x[i]);
            wall(xn, yn);
            x[i] = xn;
            y[i] = yn;
        }
        zb += zstep;
        if (a.trace != nullptr && t < a.trace_steps && mine) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = r * 32 + acc_row(half, i);
                if (row < a.n) a.trace[((size_t)col * a.trace_steps + t) * a.n + row] = x[i];
            }
        }
        put_phi(phi0 + ((t + 1) & 1) * kCols * pitch);
        __syncthreads();  // Phi of step t + 1 is complete, and everybody is done with step t's
    }

    read_out(a, r, half, lr, col, mine, x);
}

template <int PREC, int M, bool DSB, bool NOISE, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void resident_kernel(ResidentArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    resident_body<PREC, M, DSB, NOISE, WAVES == 8>(a, lds);
}

// ---------------------------------------------------------------- exact digits
//
// Discrete SB in single precision multiplies +-1 with integers.  While every
// row's weights add up to less than 2^24, no partial sum of the FP32 product
// rounds in any order, so it may be computed exactly by other means: the weights
// as base-256 digits in -128 .. 127 on the int8 matrix cores, which take 32 spins
// in half the time the FP32 MFMA needs for two.  One accumulator per objective
// goes through its digits from the highest down, shifted by eight bits between
// them; the sum is converted exactly and enters the same update.  Integers leave
// no rounding to differ: trajectories are those of the FP32 product bit for bit.
// The digits of a wave's 32 rows stream from L2 as in the other kernel, Phi
// stays in registers for the step (up to 192 spins; up to 256 it is read from LDS for
// every digit, and three digits keep 14 to 32 registers in scratch, outside the MFMAs).
// Bound by the vector instructions of the draws and the update: complete n = 100,
// m = 3, 570 000 columns with noise: 430 us per step on the FP32 product (290 of
// them MFMA, which there does not overlap with vector work), now 148.
constexpr int kDigitMax = 3;
constexpr int kDigitRegs = 8;  // groups of 32 spins whose Phi stays in registers

// groups of 32 spins in the images: past the register form an even number, the last one of zeros
__host__ __device__ constexpr int digit_groups(int n) {
    const int tiles = (n + 31) / 32;
    return tiles <= kDigitRegs ? tiles : (tiles + 1) / 2 * 2;
}

__global__ __launch_bounds__(kB) void digit_kernel(const float *__restrict__ J, int m, int Np, int n, int L,
                                                   int8_t *__restrict__ out) {
    const int tiles = (n + 31) / 32, groups = digit_groups(n);
    const int64_t idx = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (idx >= (int64_t)m * L * tiles * groups * 1024) return;
    // fragment (r, k, d, g), d = 0 the highest digit; byte j of lane (h, i) belongs to J[k][32 r + i][32 g + 16 h + j]
    const int j = (int)(idx & 15), lane = (int)(idx >> 4) & 63;
    const int64_t f = idx >> 10;
    const int g = (int)(f % groups), d = (int)(f / groups % L), k = (int)(f / groups / L % m),
              r = (int)(f / groups / L / m);
    int w = g < tiles ? (int)J[((int64_t)k * Np + 32 * r + (lane & 31)) * Np + 32 * g + 16 * (lane >> 5) + j] : 0;
    for (int e = 0; e < L - 1 - d; ++e) w = (w - (int8_t)w) >> 8;
    out[idx] = (int8_t)w;
}

// G: groups of 32 spins, the step's Phi in registers; 0: any number, read from LDS for every digit
template <int G, int L, bool NOISE>
__global__ __launch_bounds__(64 * (G == 0 ? 16 : G <= 4 ? 4 : 8), G == 5 || G == 6 ? 3 : 4) void digits_kernel(ResidentArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, half = lane >> 5, lr = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = wave % a.tiles, ct = wave / a.tiles;  // row tile, column tile of the block
    const int per_block = (int)(blockDim.x >> 6) / a.tiles, groups = G ? G : digit_groups(a.n);
    const int64_t col = ((int64_t)blockIdx.x * per_block + ct) * kCols + lr;
    const bool mine = col < a.cols;
    const int pitch = 32 * groups + 16;
    char *const phi0 = lds + (size_t)ct * 2 * kCols * pitch;
    const uint64_t g = (uint64_t)col + a.offset;
    float cf[4];
    {
        const int64_t w = mine ? col / a.R : 0;
        const double c0 = mine ? a.c0s[w] : -1.0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            cf[k] = k < a.m && c0 >= 0.0 ? (float)(-a.dt * c0 * (double)a.weights[w * a.m + k] * (double)a.jscale[k]) : 0.0f;
    }
    float x[16], y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = r * 32 + acc_row(half, i);
        const bool live = mine && row < a.n;
        x[i] = live ? init_value(a.seed, init_counter(g, a.n, row, 0), a.amp) : 0.0f;
        y[i] = live ? init_value(a.seed, init_counter(g, a.n, row, 1), a.amp) : 0.0f;
    }
    auto put_phi = [&](char *buf) __attribute__((always_inline)) {
        char *p = buf + lr * pitch + r * 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t b = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) b |= (x[4 * q + e] >= 0.0f ? 1u : 0xFFu) << (8 * e);
            *(uint32_t *)(p + acc_row(half, 4 * q)) = b;
        }
    };
    if constexpr (G == 0) {  // the padding group's Phi meets zero weights; any bytes do, but no unwritten ones
        for (int i = threadIdx.x * 4; i < per_block * 2 * kCols * pitch; i += blockDim.x * 4) *(uint32_t *)(lds + i) = 0u;
        __syncthreads();
    }
    put_phi(phi0);
    __syncthreads();
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.J, 0, a.m * L * a.tiles * groups * 1024, 0x00027000);
    const int base = r * a.m * L * groups * 1024;
    auto load_a = [&](int so) __attribute__((always_inline)) {
        return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, so, 0));
    };
    // A wave reads its fragments in order, over and over; a ring of them is in
    // flight, each slot reloaded as soon as it is used (the ring divides an
    // objective's fragments, so slots are fixed in the unrolled code).
    constexpr int RING = G == 0 ? 2 : G <= 2 ? L * G : G;
    const int end = base + a.m * L * groups * 1024;
    i32x4 av[RING];
    int so = base;
    auto next_a = [&]() __attribute__((always_inline)) {
        const i32x4 v = load_a(so);
        so += 1024;
        so = so == end ? base : so;
        return v;
    };
#pragma unroll
    for (int f = 0; f < RING; ++f) av[f] = next_a();
    constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;
    uint64_t zb = 0;
    if constexpr (NOISE)
        zb = (a.seed ^ kNoiseKey) + (g * (uint64_t)a.T * (uint64_t)a.n + (uint64_t)(r * 32 + 4 * half) + 1ull) * kGamma;
    const uint64_t zstep = (uint64_t)a.n * kGamma;

    for (int t = 0; t < a.T; ++t) {
        const float kt = a.kt_tab[t];
        const char *pc = phi0 + (t & 1) * kCols * pitch + lr * pitch + half * 16;
        float h[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) h[i] = 0.0f;
        // (seven and eight groups: 128 registers, so that two blocks share a CU, leave no room)
        constexpr bool KEEP = G > 0 && G <= 6;
        i32x4 b[KEEP ? G : 1];
        if constexpr (KEEP)
#pragma unroll
            for (int q = 0; q < G; ++q) b[q] = *(const i32x4 *)(pc + 32 * q);
#pragma unroll 1
        for (int k = 0; k < a.m; ++k) {
            const float c = k == 0 ? cf[0] : k == 1 ? cf[1] : k == 2 ? cf[2] : cf[3];
            i32x16 acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0;
#pragma unroll
            for (int d = 0; d < L; ++d) {
                if (d > 0)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[i] <<= 8;
                if constexpr (G > 0) {
#pragma unroll
                    for (int q = 0; q < G; ++q) {
                        i32x4 &v = av[(d * G + q) % RING];
                        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(v, KEEP ? b[q] : *(const i32x4 *)(pc + 32 * q), acc, 0, 0, 0);
                        v = next_a();
                        __builtin_amdgcn_sched_barrier(0x7);  // the loads stay where they are
                    }
                } else {
#pragma unroll 1
                    for (int q = 0; q < groups; q += 2) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av[e], *(const i32x4 *)(pc + 32 * (q + e)), acc,
                                                                        0, 0, 0);
                            av[e] = next_a();
                        }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) h[i] = fmaf(c, (float)acc[i], h[i]);
        }
        // Rows past n meet zero weights and are never read out: only draws of whole groups
        // of eight rows are left out, and those of four rows form one basic block.
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (NOISE && r * 32 + 8 * q >= a.n) break;
#pragma unroll
            for (int i = 4 * q; i < 4 * q + 4; ++i) {
                float yn = fmaf(kt, x[i], y[i]) + h[i];
                if constexpr (NOISE)
                    yn = fmaf(a.dt_alpha, noise_from(zb + (uint64_t)(8 * q + (i & 3)) * kGamma), yn);
                float xn = fmaf(a.dta0, yn, x[i]);
                wall(xn, yn);
                x[i] = xn;
                y[i] = yn;
            }
        }
        zb += zstep;
        if (a.trace != nullptr && t < a.trace_steps && mine) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = r * 32 + acc_row(half, i);
                if (row < a.n) a.trace[((size_t)col * a.trace_steps + t) * a.n + row] = x[i];
            }
        }
        put_phi(phi0 + ((t + 1) & 1) * kCols * pitch);
        __syncthreads();  // Phi of step t + 1 is complete, and everybody is done with step t's
    }
    read_out(a, r, half, lr, col, mine, x);
}

template <int L, bool NOISE>
void launch_digits_l(const ResidentArgs &a, hipStream_t st) {
    const int per_block = a.tiles >= 3 ? 1 : 4 / a.tiles;
    const int waves = a.tiles * per_block;
    const int64_t blocks = (a.cols + per_block * kCols - 1) / (per_block * kCols);
    QAIA_CHECK(blocks <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many replicas for the dense path");
    const size_t shmem = (size_t)per_block * 2 * kCols * (32 * digit_groups(a.n) + 16);
    static const decltype(&digits_kernel<0, L, NOISE>) kernels[] = {
        digits_kernel<0, L, NOISE>, digits_kernel<1, L, NOISE>, digits_kernel<2, L, NOISE>,
        digits_kernel<3, L, NOISE>, digits_kernel<4, L, NOISE>, digits_kernel<5, L, NOISE>,
        digits_kernel<6, L, NOISE>, digits_kernel<7, L, NOISE>, digits_kernel<8, L, NOISE>};
    hipLaunchKernelGGL(kernels[a.tiles <= kDigitRegs ? a.tiles : 0], dim3((unsigned)blocks), dim3(64 * waves), shmem, st, a);
}

void launch_digits(int L, const ResidentArgs &a, bool noise, hipStream_t st) {
    if (L == 1) noise ? launch_digits_l<1, true>(a, st) : launch_digits_l<1, false>(a, st);
    if (L == 2) noise ? launch_digits_l<2, true>(a, st) : launch_digits_l<2, false>(a, st);
    if (L == 3) noise ? launch_digits_l<3, true>(a, st) : launch_digits_l<3, false>(a, st);
}

template <int PREC, int M, bool DSB, bool NOISE>
void launch_waves(const ResidentArgs &a, hipStream_t st) {
    const int per_block = a.tiles >= 3 ? 1 : 4 / a.tiles;  // column tiles: at least three waves per block
    const int waves = a.tiles * per_block;
    const int64_t blocks = (a.cols + per_block * kCols - 1) / (per_block * kCols);
    QAIA_CHECK(blocks <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many replicas for the dense path");
    const size_t shmem = (size_t)per_block * 2 * kCols * phi_pitch<PREC>(a.n);
    if (waves <= 8)
        hipLaunchKernelGGL((resident_kernel<PREC, M, DSB, NOISE, 8>), dim3((unsigned)blocks), dim3(64 * waves), shmem, st, a);
    else
        hipLaunchKernelGGL((resident_kernel<PREC, M, DSB, NOISE, 16>), dim3((unsigned)blocks), dim3(64 * waves), shmem, st, a);
}

template <int PREC, bool DSB>
void launch_m(int m, bool noise, const ResidentArgs &a, hipStream_t st) {
    switch (m) {
#define QAIA_RES(MM)                                              \
    case MM:                                                      \
        if (noise) launch_waves<PREC, MM, DSB, true>(a, st);      \
        else launch_waves<PREC, MM, DSB, false>(a, st);           \
        break;
        QAIA_RES(1)
        QAIA_RES(2)
        QAIA_RES(3)
        QAIA_RES(4)
#undef QAIA_RES
        default: throw Error{QAIA_UNSUPPORTED, "dense path supports m <= 4"};
    }
}

}  // namespace

constexpr int kResidentMaxN = 512;

// Digits per weight of the exact product, 0 where a row's weights could add up to
// 2^24 (an FP32 partial sum may then round) or a weight needs a fourth digit.
static int digits_of(const Problem &p) {
    int64_t largest = 0;
    std::vector<int64_t> row(p.n);
    for (int k = 0; k < p.m; ++k) {
        std::fill(row.begin(), row.end(), 0);
        for (int64_t e = 0; e < p.E; ++e) {
            const int64_t w = std::llabs((long long)p.W[(size_t)k * p.E + e]);
            largest = std::max(largest, w);
            row[p.eu[e]] += w;
            row[p.ev[e]] += w;
        }
        for (const int64_t v : row)
            if (v >= (int64_t)1 << 24) return 0;
    }
    int L = 1;
    for (int64_t top = 127; top < largest; top = top * 256 + 127) ++L;
    return L <= kDigitMax ? L : 0;
}

void resident_build(Problem &p) {
    if (!p.dense.ok || p.n > kResidentMaxN) return;
    DenseImages &d = p.dense;
    const int64_t tiles = (p.n + 31) / 32;
    const int64_t e32 = p.m * tiles * kgroups<QAIA_FP32>(p.n) * 64 * 4, e16 = p.m * tiles * kgroups<QAIA_BF16>(p.n) * 64 * 8,
                  e8 = p.m * tiles * kgroups<QAIA_FP8>(p.n) * 64 * 32;
    DeviceGuard g(p.device);
    char *b = nullptr;
    d.digits = digits_of(p);
    const int64_t ed = (int64_t)p.m * d.digits * tiles * digit_groups(p.n) * 1024;
    if (!try_alloc((void **)&b, (size_t)(4 * e32 + 2 * e16 + e8 + ed))) {  // 1 KB multiples
        d.digits = 0;  // without room for the images the step kernels run
        return;
    }
    d.frag = b;
    d.F32 = (float *)b;
    d.F16 = (uint16_t *)(b + 4 * e32);
    d.F8 = (uint8_t *)(b + 4 * e32 + 2 * e16);
    d.FD = (int8_t *)(b + 4 * e32 + 2 * e16 + e8);
    auto blocks = [](int64_t n) { return dim3((unsigned)((n + kB - 1) / kB)); };
    hipLaunchKernelGGL(fragment_kernel<QAIA_FP32>, blocks(e32), dim3(kB), 0, nullptr, d.J32, p.m, d.Np, p.n, d.F32);
    hipLaunchKernelGGL(fragment_kernel<QAIA_BF16>, blocks(e16), dim3(kB), 0, nullptr, d.J16, p.m, d.Np, p.n, d.F16);
    hipLaunchKernelGGL(fragment_kernel<QAIA_FP8>, blocks(e8), dim3(kB), 0, nullptr, d.J8, p.m, d.Np, p.n, d.F8);
    if (d.digits)
        hipLaunchKernelGGL(digit_kernel, blocks(ed), dim3(kB), 0, nullptr, d.J32, p.m, d.Np, p.n, d.digits, d.FD);
    QAIA_HIP(hipGetLastError());
}

void resident_release(Problem &p) {
    DeviceGuard g(p.device);
    if (p.dense.frag) (void)hipFree(p.dense.frag);
}

bool resident_fits(const Problem &p) { return p.dense.frag != nullptr; }

void launch_resident(const Problem &p, const float *weights, int64_t W, int32_t R, const qaia_schedule &s, void *ws,
                     const WsLayout &L, uint64_t *spins, float *trace, int32_t trace_steps, hipStream_t st) {
    char *b = (char *)ws;
    ResidentArgs a{};
    a.J = s.precision == QAIA_FP32 ? (const void *)p.dense.F32
                                   : s.precision == QAIA_BF16 ? (const void *)p.dense.F16 : (const void *)p.dense.F8;
    a.weights = weights;
    a.c0s = (const double *)(b + L.c0s);
    a.kt_tab = (const float *)(b + L.kt);
    a.jscale = p.dense.scales + 8 * s.precision;
    a.dta0 = s.dt * s.a0;
    a.dt_alpha = s.dt * s.noise_alpha;
    a.amp = s.init_amp;
    a.dt = (double)s.dt;
    a.n = p.n;
    a.m = p.m;
    a.R = R;
    a.T = s.steps;
    a.tiles = (p.n + 31) / 32;
    a.cols = W * (int64_t)R;
    a.seed = s.seed;
    a.offset = s.replica_offset;
    a.spins = spins;
    a.words = p.words;
    a.trace = trace_steps > 0 ? trace : nullptr;
    a.trace_steps = trace_steps;
    const bool noise = a.dt_alpha != 0.0f, dsb = s.variant == QAIA_DSB;
    if (s.precision == QAIA_FP32 && dsb && p.dense.digits) {
        a.J = p.dense.FD;
        launch_digits(p.dense.digits, a, noise, st);
    } else if (s.precision == QAIA_FP32) {
        if (dsb) launch_m<QAIA_FP32, true>(p.m, noise, a, st);
        else launch_m<QAIA_FP32, false>(p.m, noise, a, st);
    } else if (s.precision == QAIA_BF16) {
        launch_m<QAIA_BF16, true>(p.m, noise, a, st);
    } else {
        launch_m<QAIA_FP8, true>(p.m, noise, a, st);
    }
    QAIA_HIP(hipGetLastError());
}

}  // namespace qaia
