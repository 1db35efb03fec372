// Sparse SB, one spin per lane: V replicas of one weight vector (a group) share
// a lane's neighbour list.
//
// A group's spins are spread over the NT lanes of a block, NPT spins per lane.
// Each lane keeps x and y of its spins for all V replicas, its neighbours' LDS
// places and the folded edge coefficients in registers (with four replicas and several
// spins per lane of degree past 3 the compiler puts the coefficients into scratch, 80
// to 272 bytes: it merges the last product of a chunk's two lengths, whose index then
// varies); Phi (x for ballistic
// SB, sgn x for discrete SB) of the V replicas sits in LDS as one vector per
// spin, double buffered at a fixed distance, so that a neighbour's V values
// are one read at an immediate offset: a 16-byte gather moves four replicas
// through a quarter of the LDS instructions and with fewer bank conflicts than
// four 4-byte ones, and V replicas share the addresses and coefficients.
//
// Spins take lanes in order of falling degree, so a wave's 64 spins have nearly
// equal degrees and its neighbour loop ends at the largest of them (a scalar
// branch per neighbour).  Lanes below it add 0 times a neighbour, which changes no
// value.  Groups of up to 128 spins, and up to 256 where the GPU is full and lists
// are short, run in one wave and need no barrier at all: LDS operations of a wave are
// in order.  Blocks of one wave with n <= 32 take
// several groups side by side.
//
// Every spin's update is the sequence of operations of the other sparse kernels
// (neighbours in increasing order), so results agree with theirs bit for bit.
#pragma once

#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace qaia {

typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int N> using Int = std::integral_constant<int, N>;
template <int V> struct Vec;
template <> struct Vec<1> { typedef float T; };
template <> struct Vec<4> { typedef f32x4 T; };
__device__ __forceinline__ float get(float v, int) { return v; }
__device__ __forceinline__ float get(const f32x4 &v, int i) { return v[i]; }
__device__ __forceinline__ void put(float &v, int, float x) { v = x; }
__device__ __forceinline__ void put(f32x4 &v, int i, float x) { v[i] = x; }

struct GroupArgs {
    int n, m, words, R, T, per_block, groups_per_w;
    int64_t E, groups;
    const int32_t *order, *rowptr, *col, *eid, *place, *Wt, *eu, *ev;
    const float *jcp;
    const double *c0s;
    const float *kt_tab;
    float dta0, dt_alpha, amp;
    uint64_t seed, offset;
    uint64_t *spins;
    int64_t *obj;
    float *trace;
    int trace_steps;
};

// FULL: noise injection and tracing, which keep each spin's row and counters
// in registers (V = 1).
// FLAT: the read-out of several small groups in a wave (an instance of its own: the
// place of the step loop in the code alone moves it by 2 %).
// Blocks have up to NTMAX lanes.
template <int NTMAX, int NPT, int V, int MAXDEG, bool DSB, bool FULL, bool FLAT = false>
__global__ __launch_bounds__(NTMAX) void group_kernel(GroupArgs a) {
    typedef typename Vec<V>::T VT;
    constexpr int SPAN = NTMAX * NPT;  // spins per buffer
    const int NT = NTMAX == 64 ? 64 : (int)blockDim.x;
    __shared__ __attribute__((aligned(16))) VT xs[2 * SPAN];
    __shared__ int64_t red[NTMAX / 64][V][8];
    const int n = a.n, tid = threadIdx.x, lane = tid & 63;
    const int64_t E = a.E;

    VT x[NPT], y[NPT];
    constexpr bool PACK = MAXDEG > 8;  // two 16-bit LDS places per register
    constexpr int NB = PACK ? MAXDEG / 2 : MAXDEG;
    float jv[NPT][MAXDEG];
    uint32_t nb[NPT][NB];
    int node[NPT], dw[NPT];
    bool act[NPT];
    int64_t row[NPT];    // (FULL) the spin's row
    uint64_t zb[NPT];    // (FULL) the noise stream's state at the spin's draw of step t
    constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        const int at = q * NT + tid, slot = at / n, pos = at - slot * n;
        const int64_t grp = (int64_t)blockIdx.x * a.per_block + slot;
        act[q] = slot < a.per_block && grp < a.groups;
        const int64_t w = act[q] ? grp / a.groups_per_w : 0;
        const int r0 = act[q] ? (int)(grp - w * a.groups_per_w) * V : 0;
        row[q] = w * a.R + r0;
        node[q] = act[q] ? a.order[pos] : 0;
        const int p0 = a.rowptr[node[q]], deg = act[q] ? a.rowptr[node[q] + 1] - p0 : 0;
        int wave_deg = deg;
        for (int off = 32; off > 0; off >>= 1) wave_deg = max(wave_deg, __shfl_xor(wave_deg, off));
        dw[q] = __builtin_amdgcn_readfirstlane(wave_deg);
        if constexpr (FULL)
            zb[q] = (a.seed ^ kNoiseKey) +
                    (((uint64_t)row[q] + a.offset) * (uint64_t)a.T * (uint64_t)n + (uint64_t)node[q] + 1ull) * kGamma;
#pragma unroll
        for (int d = 0; d < MAXDEG; ++d) {
            uint32_t at_d = at;
            jv[q][d] = 0.0f;
            if (d < deg) {
                at_d = slot * n + a.place[a.col[p0 + d]];
                jv[q][d] = a.jcp[w * E + a.eid[p0 + d]];
            }
            at_d *= sizeof(VT);  // bytes: at most 1024 spins of 16 bytes
            if constexpr (!PACK) nb[q][d] = at_d;
            else if (d % 2 == 0) nb[q][d / 2] = at_d;
            else nb[q][d / 2] |= at_d << 16;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint64_t g = (uint64_t)(row[q] + v) + a.offset;
            const float xv = act[q] ? init_value(a.seed, init_counter(g, n, node[q], 0), a.amp) : 0.0f;
            const float yv = act[q] ? init_value(a.seed, init_counter(g, n, node[q], 1), a.amp) : 0.0f;
            put(x[q], v, xv);
            put(y[q], v, yv);
            asm volatile("" : "+v"(x[q]), "+v"(y[q]));  // one draw after the other: interleaved, they set the register count
        }
        VT phi;
#pragma unroll
        for (int v = 0; v < V; ++v) put(phi, v, DSB ? sgn1(get(x[q], v)) : get(x[q], v));
        xs[at] = phi;
    }
    __syncthreads();  // (nothing in a block of one wave)

    auto step = [&](int t, float kt, auto buf) __attribute__((always_inline)) {
        constexpr int CUR = decltype(buf)::value;
        const char *xc = (const char *)(xs + CUR * SPAN);
        VT *xn = xs + (1 - CUR) * SPAN;
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            VT acc;
#pragma unroll
            for (int v = 0; v < V; ++v) put(acc, v, fmaf(kt, get(x[q], v), get(y[q], v)));
            // CNT neighbours from D on: all reads, then the products in order
            auto take = [&](auto from, auto cnt) __attribute__((always_inline)) {
                constexpr int D = decltype(from)::value, CNT = decltype(cnt)::value;
                VT p[CNT];
#pragma unroll
                for (int d = 0; d < CNT; ++d) {
                    // opaque: unpacked outside the loop, the places would take two registers per pair again
                    if (PACK && d % 2 == 0) asm volatile("" : "+v"(nb[q][(D + d) / 2]));
                    const uint32_t o = !PACK ? nb[q][D + d] : d % 2 == 0 ? nb[q][(D + d) / 2] & 0xffffu : nb[q][(D + d) / 2] >> 16;
                    p[d] = *(const VT *)(xc + o);
                }
#pragma unroll
                for (int d = 0; d < CNT; ++d)
#pragma unroll
                    for (int v = 0; v < V; ++v) put(acc, v, fmaf(jv[q][D + d], get(p[d], v), get(acc, v)));
            };
            if constexpr (MAXDEG == 3) {
                if (dw[q] == 3) take(Int<0>{}, Int<3>{});
                else if (dw[q] == 2) take(Int<0>{}, Int<2>{});
                else if (dw[q] == 1) take(Int<0>{}, Int<1>{});
            } else {
                auto chunk = [&](auto from) __attribute__((always_inline)) {
                    const int left = dw[q] - decltype(from)::value;
                    if (left > 2) take(from, Int<4>{});
                    else if (left > 0) take(from, Int<2>{});
                };
                // Eight neighbours: one replica is bound by the reads' latency, so more of them go
                // at once (113 nodes of degree up to 14, 784 replicas, 200 steps 161 -> 126 us;
                // 300 nodes of up to 27 with noise, 1600 replicas 1136 -> 899).
                auto chunks = [&](auto from) __attribute__((always_inline)) {
                    constexpr int D = decltype(from)::value;
                    if (V == 1 && dw[q] - D > 4) {
                        take(from, Int<8>{});
                    } else {
                        chunk(from);
                        if (V > 1) chunk(Int<D + 4>{});
                    }
                };
                chunks(Int<0>{});
                if constexpr (MAXDEG > 8) {
                    if (dw[q] > 8) chunks(Int<8>{});
                    if (dw[q] > 16) {
                        chunks(Int<16>{});
                        chunks(Int<24>{});
                    }
                }
            }
            if constexpr (FULL) {
                if (a.dt_alpha != 0.0f && act[q]) put(acc, 0, fmaf(a.dt_alpha, noise_from(zb[q]), get(acc, 0)));
                zb[q] += (uint64_t)n * kGamma;
            }
            VT phi;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                float yn = get(acc, v), xv = fmaf(a.dta0, yn, get(x[q], v));
                wall(xv, yn);
                put(x[q], v, xv);
                put(y[q], v, yn);
                put(phi, v, DSB ? sgn1(xv) : xv);
            }
            xn[q * NT + tid] = phi;
            if constexpr (FULL)
                if (a.trace != nullptr && t < a.trace_steps && act[q])
                    a.trace[(row[q] * a.trace_steps + t) * n + node[q]] = get(x[q], 0);
        }
        if constexpr (NTMAX > 64) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
    };
    // The step coefficients come 64 at a time through vector loads, the next 64
    // under way during the current: scalar loads share the counter that the LDS
    // reads wait on and return out of order, so each would stall them.
    float knext = a.kt_tab[min(lane, a.T - 1)];
    for (int t0 = 0; t0 < a.T; t0 += 64) {
        const float kcur = knext;
        knext = a.kt_tab[min(t0 + 64 + lane, a.T - 1)];
        auto coef = [&](int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(kcur), i)); };
        const int cnt = min(64, a.T - t0);
        int i = 0;
        for (; i + 1 < cnt; i += 2) {
            step(t0 + i, coef(i), Int<0>{});
            step(t0 + i + 1, coef(i + 1), Int<1>{});
        }
        if (i < cnt) step(t0 + i, coef(i), Int<0>{});
    }
    __syncthreads();

    // signs in node order: word of 64 spins by ballot needs node order, so they go through LDS once more
#pragma unroll
    for (int q = 0; q < NPT; ++q)
        if (act[q]) {
            VT s;
#pragma unroll
            for (int v = 0; v < V; ++v) put(s, v, get(x[q], v) < 0.0f ? -1.0f : 1.0f);
            xs[(q * NT + tid) / n * n + node[q]] = s;
        }
    __syncthreads();
    if constexpr (FLAT) {  // a lane per (replica, objective) walks the edges
        const float *xf = (const float *)xs;
        for (int i = tid; i < a.per_block * V * a.m; i += NT) {
            const int sr = i / a.m, k = i - sr * a.m, slot = sr / V, v = sr - slot * V;
            const int64_t grp = (int64_t)blockIdx.x * a.per_block + slot;
            if (grp >= a.groups) break;
            const int64_t w = grp / a.groups_per_w;
            const int r = (int)(grp - w * a.groups_per_w) * V + v;
            if (r >= a.R) continue;
            const bool valid = a.c0s[w] >= 0.0;
            const float *s = xf + slot * n * V + v;
            int64_t cut = 0;
#pragma unroll 4
            for (int64_t e = 0; e < E; ++e)
                cut += s[a.eu[e] * V] != s[a.ev[e] * V] ? (int64_t)a.Wt[(int64_t)k * E + e] : 0;
            a.obj[(w * a.R + r) * a.m + k] = valid ? cut : 0;
            if (k == 0) {
                uint64_t bits = 0;
#pragma unroll 4
                for (int j = 0; j < n; ++j) bits |= (uint64_t)(s[j * V] < 0.0f) << j;
                a.spins[w * a.R + r] = valid ? bits : 0ull;
            }
        }
        return;
    }
    for (int slot = 0; slot < a.per_block; ++slot) {
        const int64_t grp = (int64_t)blockIdx.x * a.per_block + slot;
        if (grp >= a.groups) break;
        const int64_t w = grp / a.groups_per_w;
        const int r0 = (int)(grp - w * a.groups_per_w) * V, count = min(V, a.R - r0);
        const int64_t first = w * a.R + r0;
        const bool valid = a.c0s[w] >= 0.0;
        const VT *s = xs + slot * n;
        for (int wd = tid >> 6; wd < a.words; wd += NT / 64) {
            const int i = wd * 64 + lane;
            VT sv;
#pragma unroll
            for (int v = 0; v < V; ++v) put(sv, v, 1.0f);
            if (i < n) sv = s[i];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const uint64_t bits = __ballot(get(sv, v) < 0.0f);
                if (lane == 0 && v < count) a.spins[(first + v) * a.words + wd] = valid ? bits : 0ull;
            }
        }
        // exact cuts, Eq. (1): lanes stride the edges for all replicas of the group,
        // one objective at a time (all of them at once set the register count)
        for (int k = 0; k < a.m; ++k) {
            int64_t acc[V];
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = 0;
            if (valid)
                for (int64_t e = tid; e < E; e += NT) {
                    const VT su = s[a.eu[e]], sv = s[a.ev[e]];
                    const int64_t wt = a.Wt[(int64_t)k * E + e];
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] += get(su, v) != get(sv, v) ? wt : 0;
                }
#pragma unroll
            for (int v = 0; v < V; ++v) {
                int64_t c = acc[v];
                for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
                if (lane == 0) red[tid >> 6][v][k] = c;
            }
        }
        __syncthreads();
        for (int i = tid; i < count * a.m; i += NT) {
            const int v = i / a.m, k = i - v * a.m;
            int64_t c = 0;
            for (int wv = 0; wv < NT / 64; ++wv) c += red[wv][v][k];
            a.obj[(first + v) * a.m + k] = c;
        }
        __syncthreads();  // red is rewritten by the next slot
    }
}

// One of the launches of group.hip: NTMAX x NPT lanes x spins, V replicas.  LONG: shapes
// that lists of more than eight neighbours take.
template <int NTMAX, int NPT, int V, bool DSB, bool FULL, bool LONG>
void launch_group_deg(int maxdeg, bool flat, dim3 grid, dim3 block, const GroupArgs &a, hipStream_t st) {
    if constexpr (NTMAX == 64 && NPT == 1)
        if (flat) {
            if (maxdeg <= 3) hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 3, DSB, FULL, true>), grid, block, 0, st, a);
            else if (maxdeg <= 8) hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 8, DSB, FULL, true>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 32, DSB, FULL, true>), grid, block, 0, st, a);
            return;
        }
    if (maxdeg <= 3) hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 3, DSB, FULL>), grid, block, 0, st, a);
    else if (maxdeg <= 8) hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 8, DSB, FULL>), grid, block, 0, st, a);
    else if constexpr (LONG) hipLaunchKernelGGL((group_kernel<NTMAX, NPT, V, 32, DSB, FULL>), grid, block, 0, st, a);
    else throw Error{QAIA_DEVICE_ERROR, "no kernel of this shape for so many neighbours"};  // group_shape picks none
}

void launch_group_v1(int shape, bool dsb, int maxdeg, bool flat, dim3 grid, dim3 block, const GroupArgs &a, hipStream_t st);
void launch_group_full(int shape, bool dsb, int maxdeg, bool flat, dim3 grid, dim3 block, const GroupArgs &a, hipStream_t st);

}  // namespace qaia
