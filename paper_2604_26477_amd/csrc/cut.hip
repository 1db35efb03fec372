// Exact cut evaluation of dense graphs on the matrix cores, Eq. (1).
//
// With s in {-1, +1}^n, C_k(s) = (T_k - Q_k) / 2 with T_k = sum_E W_k and
// Q_k = sum_{u < v} W_k,uv s_u s_v = sum_u s_u (U_k s)_u, U_k the strict upper
// triangle.  W_k is split into signed base-256 digits, W = sum_l 256^l d_l with
// d_l in [-128, 127], so that every product d_l s is an int8 matrix product with
// exact int32 sums (|sum| <= 128 n); the digits are put together in int64.
// Whole numbers throughout: the result is that of the sum over cut edges.
//
// The "slices" are the S = m L digit matrices (L = digits that the largest
// weight needs: 3 for N(0,1) weights at 16 fraction bits).  Their images hold
// the MFMA A operands as the instruction reads them: tile (r, g) of a slice is
// 64 lanes x 16 bytes, lane (h, i) holding rows 32 r + i, spins 32 g + 16 h ..
// + 15; the B operand has the same spins per lane, so any internal order of the
// instruction pairs them.
//
// A block of four waves takes 128 samples (four 32-column B tiles) and one chunk
// of up to 448 spins, whose bits it expands to int8 in LDS in operand order.  Its
// waves take (row tile, three slices) items: three accumulators per column tile
// (192 registers, two waves per SIMD), so that an A tile read from L2 serves four
// MFMAs and a B tile read from LDS three: at 32 cycles per MFMA the 64 bytes per
// cycle of the vector cache and the 128 of the LDS are half used.  Only tiles on
// or above the diagonal are visited.  The epilogue multiplies by the row spins
// (one operation per element, shared by the slices, and one per slice) and adds
// the digits to int64 sums in LDS.  570 000 samples of a complete 200-node graph,
// m = 3, 19 900 edges: 4.37 ms walking the edges, 0.20 ms here (matrix cores 29 %
// busy, vector units 30 %; 0.23 ms with an item's first A tiles and row spins
// read when it begins); 4096 samples at 2048 nodes: 5.06 and 0.10 ms.  Two column
// tiles per wave and four waves per SIMD instead: 0.31 ms.
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace qaia {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int kB = 256;
constexpr int kCols = 128;       // samples per block
constexpr int kChunkTiles = 14;  // 32-spin tiles per chunk: 56 KB of int8 spins, 7 KB of spin words, 8 KB of sums at m = 8
constexpr int kGroup = 3;        // slices per item

// One thread per (edge, objective): the digits of its weight into the upper
// triangle's images.
__global__ __launch_bounds__(kB) void cut_image_kernel(const int32_t *__restrict__ eu, const int32_t *__restrict__ ev,
                                                       const int32_t *__restrict__ Wt, int64_t E, int m, int L, int T,
                                                       int8_t *__restrict__ img) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= E * m) return;
    const int k = (int)(i / E);
    const int64_t e = i - (int64_t)k * E;
    const int u = eu[e], v = ev[e];
    const int64_t tile = ((int64_t)(u >> 5) * T + (v >> 5)) * 1024;
    const int at = ((((v >> 4) & 1) * 32) + (u & 31)) * 16 + (v & 15);
    int64_t w = Wt[i];
    for (int l = 0; l < L; ++l) {
        const int8_t d = (int8_t)(w & 255);
        w = (w - d) >> 8;
        img[(int64_t)(k * L + l) * T * T * 1024 + tile + at] = d;
    }
}

__global__ __launch_bounds__(kB) void cut_zero_kernel(uint4 *__restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kB)
        p[i] = make_uint4(0, 0, 0, 0);
}

// four spin bits -> four int8 spins: +1 for a clear bit, -1 for a set one
__device__ __forceinline__ int spins4(uint32_t nibble) {
    const uint32_t spread = (uint32_t)__umul24(nibble, 0x00204081u) & 0x01010101u;
    return (int)(((spread << 8) - spread) | 0x01010101u);
}

struct CutArgs {
    const uint32_t *spins;  // 32-bit words, 2 * words per sample
    int64_t count;
    int words2, m, L, T, parts;
    const int8_t *img;
    const int64_t *total;
    int64_t *obj;
};

// SINGLE: one block sees all of its samples' tiles and writes the cuts;
// otherwise the blocks add their shares of Q to obj.
template <bool SINGLE>
__global__ __launch_bounds__(kB, 2) void cut_kernel(CutArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, lr = lane & 31;
    const int T = a.T, S = a.m * a.L, G = (S + kGroup - 1) / kGroup;
    const int kc = blockIdx.y / a.parts, part = blockIdx.y - kc * a.parts;
    const int g0 = kc * kChunkTiles, g1 = min(T, g0 + kChunkTiles);  // the chunk's spin tiles
    const int64_t col0 = (int64_t)blockIdx.x * kCols;
    unsigned long long *q = (unsigned long long *)lds;  // [m][kCols]
    uint32_t *words = (uint32_t *)(q + a.m * kCols);       // [chunk tile][kCols]: the spins as they came
    i32x4 *bs = (i32x4 *)(words + (g1 - g0) * kCols);      // [chunk tile][column tile][lane]
    for (int i = threadIdx.x; i < a.m * kCols; i += kB) q[i] = 0ull;
    for (int f = wave; f < (g1 - g0) * 4; f += kB / 64) {
        const int64_t col = col0 + (f & 3) * 32 + lr;
        const uint32_t w = col < a.count ? a.spins[col * a.words2 + g0 + (f >> 2)] : 0u;
        if (half == 0) words[(f >> 2) * kCols + (f & 3) * 32 + lr] = w;
        i32x4 b;
#pragma unroll
        for (int d = 0; d < 4; ++d) b[d] = spins4(__builtin_amdgcn_ubfe(w, 16 * half + 4 * d, 4));
        bs[f * 64 + lane] = b;
    }
    __syncthreads();
    const bool one = a.L == kGroup;
    const int rows = min(T, g1);  // row tiles with something on or above the diagonal
    // Items (row tile, group) in row-major order, every (4 parts)-th one.  One loop
    // over all their tiles: an item's last tile loads the first A tiles of the
    // wave's next item, which arrive behind the sums.
    const int step = 4 * a.parts, items = rows * G;
    int item = part * 4 + wave;
    if (item < items) {
        int r = item / G, grp = item - r * G, g = max(r, g0);
        i32x4 av[kGroup];
        i32x16 acc[kGroup][4];
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.img, 0, S * T * T * 1024, 0x00027000);
        auto load = [&](int s, int rr, int gg, int g) __attribute__((always_inline)) {
            // (a missing slice reads the last one; its sums are dropped)
            const int at = ((min(gg * kGroup + s, S - 1) * T + rr) * T + g) * 1024;
            return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, at, 0));
        };
#pragma unroll
        for (int s = 0; s < kGroup; ++s) {
            av[s] = load(s, r, grp, g);
            asm volatile("" : "+v"(av[s]));  // arrived: otherwise the loop's first use would wait for its own loads
        }
        bool first = true;
        for (;;) {
            const bool last = g + 1 == g1;
            const int ni = last && item + step < items ? item + step : item;
            const int nr = ni / G, ng = last ? max(nr, g0) : g + 1;
            i32x4 bv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) bv[c] = bs[((g - g0) * 4 + c) * 64 + lane];
            // each A tile is replaced as soon as its MFMAs are under way
            auto tile = [&](auto zero) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < kGroup; ++s) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        i32x16 z = {};
                        acc[s][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av[s], bv[c], decltype(zero)::value ? z : acc[s][c],
                                                                         0, 0, 0);
                    }
                    av[s] = load(s, nr, ni - nr * G, ng);
                    __builtin_amdgcn_sched_barrier(0x7);
                }
            };
            if (first) tile(std::true_type{});
            else tile(std::false_type{});
            if (last) {
                const int s0 = grp * kGroup, ns = min(kGroup, S - s0);
                // this lane's columns' spins of the row tile
                uint32_t rw[4];
                if (r >= g0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) rw[c] = words[(r - g0) * kCols + c * 32 + lr] >> (4 * half);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int64_t col = min(col0 + c * 32 + lr, a.count - 1);
                        rw[c] = a.spins[col * a.words2 + r] >> (4 * half);
                    }
                }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // -x = ~x + 1: the row signs as an exclusive or (one v_xad per slice), the ones added at the end
            const int ones = __popc(rw[c] & 0x0f0f0f0fu);
            int sum[kGroup] = {ones, ones, ones};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // accumulator slot i holds row (i / 4) * 8 + half * 4 + i % 4
                const int neg = __builtin_amdgcn_sbfe((int)rw[c], (i >> 2) * 8 + (i & 3), 1);
#pragma unroll
                for (int s = 0; s < kGroup; ++s) sum[s] += acc[s][c][i] ^ neg;
            }
            unsigned long long *qc = q + c * 32 + lr;
            if (one) {  // the item holds one objective's three digits
                const int64_t v = (int64_t)sum[0] + ((int64_t)sum[1] << 8) + ((int64_t)sum[2] << 16);
                atomicAdd(qc + grp * kCols, (unsigned long long)v);
                continue;
            }
#pragma unroll
            for (int s = 0; s < kGroup; ++s)
                if (s < ns) {
                    const int k = (s0 + s) / a.L, l = s0 + s - k * a.L;
                    atomicAdd(qc + k * kCols, (unsigned long long)((int64_t)sum[s] << (8 * l)));
                }
        }
                if (ni == item) break;
                item = ni;
                r = nr;
                grp = ni - nr * G;
            }
            first = last;
            g = ng;
        }
    }
    __syncthreads();
    const int64_t col = col0 + (threadIdx.x & (kCols - 1));
    if (col >= a.count) return;
    for (int k = threadIdx.x / kCols; k < a.m; k += kB / kCols) {
        const int64_t Q = (int64_t)q[k * kCols + (threadIdx.x & (kCols - 1))];
        int64_t *out = a.obj + col * a.m + k;
        if (SINGLE) *out = (a.total[k] - Q) >> 1;  // T and Q have the same parity
        else atomicAdd((unsigned long long *)out, (unsigned long long)Q);
    }
}

__global__ __launch_bounds__(kB) void cut_clear_kernel(int64_t *__restrict__ obj, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) obj[i] = 0;
}

__global__ __launch_bounds__(kB) void cut_finish_kernel(int64_t *__restrict__ obj, int64_t n, int m,
                                                        const int64_t *__restrict__ total) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) obj[i] = (total[i % m] - obj[i]) >> 1;
}

// Digits that hold every weight: L balanced base-256 digits hold -128 u .. 127 u
// with u = (256^L - 1) / 255.
int digits_for(const std::vector<int32_t> &W) {
    int32_t lo = 0, hi = 0;
    for (int32_t w : W) {
        lo = std::min(lo, w);
        hi = std::max(hi, w);
    }
    int L = 1;
    for (int64_t u = 1; (int64_t)hi > 127 * u || (int64_t)lo < -128 * u; u = 256 * u + 1) ++L;
    return L;
}

}  // namespace

// Built where the matrix form does less work than a walk over the edges: at S = 9 the
// walk's instructions per edge and the MFMAs' cycles per pair of spins are even at a
// density near 2 %, and the line is drawn at 1/32 of the pairs.  Walk against matrices
// there: 129 nodes, m = 4, 10 000 samples 93 / 15 us, 570 000 244 / 143; 1024 nodes, m = 3,
// 10 000 124 / 66; 73 nodes of degree 3, m = 4, 10 000 29 / 15, 570 000 75 / 79, which is why
// launch_evaluate still walks the edges of small graphs for many samples.  Images of at
// most 512 MiB.
void cut_build(Problem &p) {
    CutImages &c = p.cut;
    if (p.E < 64 || p.E < (int64_t)p.n * p.n / 64) return;
    const int64_t T = (p.n + 31) / 32;
    const int L = digits_for(p.W);
    const int64_t bytes = (int64_t)p.m * L * T * T * 1024;
    if (bytes > (int64_t(1) << 29)) return;
    DeviceGuard g(p.device);
    // without room for the images the edges are walked
    if (!try_alloc((void **)&c.img, (size_t)bytes)) return;
    if (!try_alloc((void **)&c.total, sizeof(int64_t) * (size_t)p.m)) {
        (void)hipFree(c.img);
        c.img = nullptr;
        return;
    }
    QAIA_HIP(hipMemcpy(c.total, p.total.data(), sizeof(int64_t) * (size_t)p.m, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(cut_zero_kernel, dim3((unsigned)std::min<int64_t>((bytes / 16 + kB - 1) / kB, 4096)), dim3(kB), 0,
                       nullptr, (uint4 *)c.img, bytes / 16);
    const int64_t n = p.E * p.m;
    hipLaunchKernelGGL(cut_image_kernel, dim3((unsigned)((n + kB - 1) / kB)), dim3(kB), 0, nullptr, p.d_eu, p.d_ev, p.d_W,
                       p.E, p.m, L, (int)T, c.img);
    QAIA_HIP(hipGetLastError());
    c.T = (int)T;
    c.L = L;
    c.ok = true;
}

void cut_release(Problem &p) {
    DeviceGuard g(p.device);
    if (p.cut.img) (void)hipFree(p.cut.img);
    if (p.cut.total) (void)hipFree(p.cut.total);
}

void launch_cut(const Problem &p, const uint64_t *spins, int64_t count, int64_t *obj, hipStream_t st) {
    const CutImages &c = p.cut;
    const int64_t bx = (count + kCols - 1) / kCols;
    QAIA_CHECK(bx <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many samples");
    const int chunks = (c.T + kChunkTiles - 1) / kChunkTiles;
    const int G = (p.m * c.L + kGroup - 1) / kGroup;
    // about 1024 blocks where there are too few samples to fill the GPU, four items (one per wave) each at least
    const int64_t most = std::max<int64_t>(1, (int64_t)std::min(c.T, kChunkTiles) * G / 4);
    const int parts = (int)std::min<int64_t>(most, std::max<int64_t>(1, 1024 / (bx * chunks)));
    const size_t shmem = (size_t)p.m * kCols * 8 + (size_t)std::min(c.T, kChunkTiles) * (4096 + kCols * 4);
    const CutArgs a{(const uint32_t *)spins, count, 2 * p.words, p.m, c.L, c.T, parts, c.img, c.total, obj};
    const dim3 grid((unsigned)bx, (unsigned)(chunks * parts));
    if (chunks * parts == 1) {
        hipLaunchKernelGGL(cut_kernel<true>, grid, dim3(kB), shmem, st, a);
    } else {
        const int64_t n = count * p.m;
        const dim3 flat((unsigned)((n + kB - 1) / kB));
        hipLaunchKernelGGL(cut_clear_kernel, flat, dim3(kB), 0, st, obj, n);
        hipLaunchKernelGGL(cut_kernel<false>, grid, dim3(kB), shmem, st, a);
        hipLaunchKernelGGL(cut_finish_kernel, flat, dim3(kB), 0, st, obj, n, p.m, c.total);
    }
    QAIA_HIP(hipGetLastError());
}

}  // namespace qaia
