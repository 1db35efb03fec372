// Non-dominated filtering of a sample pool (section "Pareto filtering",
// dominance of Eq. 4 in cut / maximisation space) with duplicate merging.
// A sampler's pool repeats the same cuts many times (at the 42-node
// four-objective workload, 10.24 M rows hold about sixteen thousand distinct
// vectors), so duplicates go first, and what is left is usually short enough
// to compare every pair.
//
// 1. Duplicate merging.  Every row looks its vector up in an open-addressing
//    hash table; each distinct vector ends with one slot holding its smallest
//    sample index (the representative).  Rows are first merged per chunk of
//    1008 in an LDS table, so that only each chunk's distinct vectors reach
//    the global one.  The occupied slots are collected into the list of distinct vectors
//    (in no particular order; nothing below needs one).
// 2. Lists longer than kPairMax only: pivots and pruning.  On an evenly
//    strided sample of the list, the row with the largest normalised weighted
//    sum is taken for each of 256 fixed positive directions (a maximiser of a
//    positive weighted sum is non-dominated, so the pivots sit on or near the
//    front), and a row is dropped when some other pivot is >= it
//    componentwise.  If more than kPairMax rows are left, each chunk of 1024
//    then drops the rows that another row of the chunk dominates.  Both only
//    drop dominated rows, and every dominated row keeps a dominator (a front
//    vector above it is never dropped), so the rest has the pool's front.
// 3. Packing.  The listed vectors as 32-bit offsets from the first one, in
//    list order; offsets that do not fit raise a flag.  A list that is still
//    longer than kPairMax is laid out by falling value of a monotone key in
//    kBuckets steps, so that a row's dominators stand before the end of its step.
// 4. Pairs.  Every pair of 256-row tiles is one work item of a persistent
//    grid: a row is marked when another row is >= it componentwise (the
//    vectors are distinct, so that is dominance).  Of an ordered list only the
//    tiles before the end of the row's step are compared.
// 5. The unmarked rows' sample indices go into a bitmap over 0..M-1 and are
//    emitted in ascending order.
// Nothing is sorted: a sort by objective costs three launches per digit, all
// of which must be queued before the list length is known (96 launches, 0.5 ms
// of the 1.1 ms that the headline pool took), to save half of the comparisons
// (10 us of them).
// The non-dominated ranks sort every row lexicographically descending (no
// merging or pruning; equal vectors become adjacent, smallest index first, and
// the first of each run represents it), a linear extension of dominance, and
// peel the unique list with order-dependent passes: within chunks of 1024, a
// row is dropped when an earlier one is >= it, then survivors against earlier
// survivors; at most kPairMax rows take tile pairs (it <= jt) instead.
// Every step runs on the caller's stream and every count stays on the device
// (launches that the list length does not need return at once).
#include <climits>
#include <type_traits>

#include "radix.hpp"

namespace qaia {

namespace {

constexpr int kB = 256;
constexpr int kChunk = 1024;
constexpr int kDirs = 256;          // pivot directions
constexpr int kSampleRows = 1 << 17;  // rows of the pivot sample (at most)
constexpr int kCandBlocks = 512;     // blocks of the pivot search (at most)
// Longest list that goes to the pair pass as it is: at 20 000 vectors of four
// objectives (the headline pool) its 4e8 pairs take 0.1 ms, and pruning first
// left 16 700 of them, which saved less than its own kernels took.
constexpr int64_t kPairMax = 1 << 15;
constexpr int kPairBlocks = 2048;      // persistent grid of the pair pass

unsigned grid_for_n(int64_t n, int per) {
    const int64_t g = (n + per - 1) / per;
    return (unsigned)(g > 1 ? g : 1);
}

__global__ void fill_u8_kernel(uint8_t *p, int64_t n, uint8_t v) {
    int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void fill_i64_kernel(int64_t *p, int64_t n, int64_t v) {
    int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) p[i] = v;
}

// lo[k] = INT64_MAX, hi[k] = INT64_MIN for the range reductions
__global__ void range_init_kernel(int64_t *lo, int64_t *hi, int n) {
    if ((int)threadIdx.x < n) {
        lo[threadIdx.x] = INT64_MAX;
        hi[threadIdx.x] = INT64_MIN;
    }
}

// Fixed positive direction d over m objectives: exponential variates of a
// counter hash, i.e. a Dirichlet(1, ..., 1) draw (only their spread over the
// simplex matters).
__device__ __forceinline__ float direction(int d, int k) {
    uint64_t z = ((uint64_t)d << 8 | (uint64_t)k) * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    const float u = ((float)(z >> 40) + 0.5f) * (1.0f / 16777216.0f);
    return -__logf(u);
}

// A row list: position i < n names row list[i] (the identity without a list);
// n is read from device memory when d_n is given.
struct RowList {
    const int32_t *list;
    const int64_t *d_n;
    int64_t n_host;
    __device__ __forceinline__ int64_t n() const { return d_n ? *d_n : n_host; }
    __device__ __forceinline__ int64_t row(int64_t i) const { return list ? (int64_t)list[i] : i; }
};

// The pivot sample: positions s * stride, s < ns, stride = ceil(n / kSampleRows).
__device__ __forceinline__ void sample_plan(int64_t n, int64_t &stride, int64_t &ns) {
    stride = n > kSampleRows ? (n + kSampleRows - 1) / kSampleRows : 1;
    ns = (n + stride - 1) / stride;
}

// Per-objective range of the sample rows (SAMPLE; lists of at most kPairMax
// rows are not pruned and need none) or of every row.
template <int MM, bool SAMPLE>
__global__ __launch_bounds__(kB) void sample_range_kernel(const int64_t *__restrict__ obj, RowList L,
                                                          int64_t *__restrict__ lo, int64_t *__restrict__ hi) {
    __shared__ int64_t rl[MM][kB], rh[MM][kB];
    int64_t stride = 1, ns = L.n();
    if (SAMPLE) {
        if (ns <= kPairMax) return;
        sample_plan(L.n(), stride, ns);
    }
    int64_t a[MM], b[MM];
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        a[k] = INT64_MAX;
        b[k] = INT64_MIN;
    }
    for (int64_t s = (int64_t)blockIdx.x * kB + threadIdx.x; s < ns; s += (int64_t)gridDim.x * kB) {
        const int64_t *y = obj + L.row(s * stride) * MM;
#pragma unroll
        for (int k = 0; k < MM; ++k) {
            a[k] = min(a[k], y[k]);
            b[k] = max(b[k], y[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        rl[k][threadIdx.x] = a[k];
        rh[k][threadIdx.x] = b[k];
    }
    __syncthreads();
    for (int s = kB / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
#pragma unroll
            for (int k = 0; k < MM; ++k) {
                rl[k][threadIdx.x] = min(rl[k][threadIdx.x], rl[k][threadIdx.x + s]);
                rh[k][threadIdx.x] = max(rh[k][threadIdx.x], rh[k][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if ((int)threadIdx.x < MM) {
        atomicMin((long long *)&lo[threadIdx.x], (long long)rl[threadIdx.x][0]);
        atomicMax((long long *)&hi[threadIdx.x], (long long)rh[threadIdx.x][0]);
    }
}

// Block b scans its share of the sample; thread d keeps the best row of
// direction d (largest score, then smallest row index) and offers it to
// best[d] as (score bits, ~row): scores are >= 0, so their bits order them.
template <int MM>
__global__ __launch_bounds__(kB) void pivot_cand_kernel(const int64_t *__restrict__ obj, RowList L,
                                                        const int64_t *__restrict__ lo, const int64_t *__restrict__ hi,
                                                        unsigned long long *__restrict__ best_of) {
    __shared__ float yn[kB][MM];
    __shared__ int32_t yi[kB];
    if (L.n() <= kPairMax) return;
    int64_t stride, ns;
    sample_plan(L.n(), stride, ns);
    float w[MM];
    float scale[MM];
    double off[MM];
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        w[k] = direction(threadIdx.x, k);
        off[k] = (double)lo[k];
        const double span = (double)hi[k] - (double)lo[k];
        scale[k] = span > 0.0 ? (float)(1.0 / span) : 0.0f;
    }
    float best = -1.0f;
    int32_t bidx = INT32_MAX;
    const int64_t per = (ns + gridDim.x - 1) / gridDim.x;
    const int64_t s0 = (int64_t)blockIdx.x * per, s1 = min(ns, s0 + per);
    for (int64_t c = s0; c < s1; c += kB) {
        const int64_t s = c + threadIdx.x;
        if (s < s1) {
            const int64_t r = L.row(s * stride);
#pragma unroll
            for (int k = 0; k < MM; ++k) yn[threadIdx.x][k] = (float)(((double)obj[r * MM + k] - off[k]) * scale[k]);
            yi[threadIdx.x] = (int32_t)r;
        }
        __syncthreads();
        const int cnt = (int)min<int64_t>(kB, s1 - c);
        for (int t = 0; t < cnt; ++t) {
            float sc = 0.0f;
#pragma unroll
            for (int k = 0; k < MM; ++k) sc = fmaf(w[k], yn[t][k], sc);
            if (sc > best || (sc == best && yi[t] < bidx)) {
                best = sc;
                bidx = yi[t];
            }
        }
        __syncthreads();
    }
    if (best >= 0.0f)
        atomicMax(&best_of[threadIdx.x],
                  ((unsigned long long)__float_as_uint(best) << 32) | (uint32_t)~(uint32_t)bidx);
}

// Appends `value` of the lanes with `mine` to out[*count ..], one atomic per wave.
template <typename T>
__device__ __forceinline__ void wave_append(bool mine, T value, T *__restrict__ out, int64_t *__restrict__ count) {
    const uint64_t mask = __ballot(mine);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63, leader = __ffsll((unsigned long long)mask) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd((unsigned long long *)count, (unsigned long long)__popcll(mask));
    base = __shfl(base, leader);
    if (mine) out[base + __popcll(mask & ((1ull << lane) - 1ull))] = value;
}

// Appends the listed rows that no pivot dominates.  A block takes 64 rows at a
// time and each of its four waves a quarter of the pivots, so that a list of a
// few ten thousand rows fills the GPU.
template <int MM>
__global__ __launch_bounds__(kB) void prune_kernel(const int64_t *__restrict__ obj, RowList L,
                                                   const unsigned long long *__restrict__ best_of,
                                                   int32_t *__restrict__ out, int64_t *__restrict__ count) {
    __shared__ int64_t pv[kDirs][MM];
    __shared__ uint64_t hit[kB / 64];
    const int64_t n = L.n();
    if (n <= kPairMax) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // (a row may be the pivot of several directions)
    const int32_t mine = (int32_t)~(uint32_t)best_of[threadIdx.x];
#pragma unroll
    for (int k = 0; k < MM; ++k) pv[threadIdx.x][k] = obj[(int64_t)mine * MM + k];
    __syncthreads();
    const int p0 = wave * 64, p1 = p0 + 64;
    for (int64_t c = (int64_t)blockIdx.x * 64; c < n; c += (int64_t)gridDim.x * 64) {
        const int64_t i = c + lane;
        const bool live = i < n;
        const int64_t r = live ? L.row(i) : 0;
        int64_t y[MM];
#pragma unroll
        for (int k = 0; k < MM; ++k) y[k] = live ? obj[r * MM + k] : 0;
        bool drop = !live;
        for (int p = p0; p < p1; ++p) {
            bool ge = true, ne = false;  // the listed vectors are distinct: an equal pivot is the row itself
#pragma unroll
            for (int k = 0; k < MM; ++k) {
                ge &= pv[p][k] >= y[k];
                ne |= pv[p][k] != y[k];
            }
            drop |= ge && ne;
            if ((p & 7) == 7 && __ballot(!drop) == 0) break;
        }
        const uint64_t dropped = __ballot(drop);
        if (lane == 0) hit[wave] = dropped;
        __syncthreads();
        if (wave == 0) {
            uint64_t all = 0;
            for (int w = 0; w < kB / 64; ++w) all |= hit[w];
            wave_append(((all >> lane) & 1ull) == 0, (int32_t)r, out, count);
        }
        __syncthreads();
    }
}

// Clears what a filter call starts from: the hash table (-1, sixteen bytes a
// store), the bitmap of kept rows, the counts, the pivots and the sample range.
__global__ __launch_bounds__(kB) void filter_init_kernel(int4 *__restrict__ table, int64_t table_quads,
                                                         uint32_t *__restrict__ bits, int64_t words,
                                                         int64_t *__restrict__ counts,
                                                         unsigned long long *__restrict__ best_of,
                                                         int64_t *__restrict__ lo, int64_t *__restrict__ hi) {
    const int64_t t0 = (int64_t)blockIdx.x * kB + threadIdx.x, step = (int64_t)gridDim.x * kB;
    for (int64_t i = t0; i < table_quads; i += step) table[i] = make_int4(-1, -1, -1, -1);
    for (int64_t i = t0; i < words; i += step) bits[i] = 0u;
    if (blockIdx.x == 0) {
        best_of[threadIdx.x] = 0ull;
        if (threadIdx.x < 8) {
            counts[threadIdx.x] = 0;
            lo[threadIdx.x] = INT64_MAX;
            hi[threadIdx.x] = INT64_MIN;
        }
    }
}

// 32-bit hash of a vector: a multiply for each of the two words of an objective
// and a final mix (32-bit multiplies issue at a quarter of the rate, 64-bit ones
// take three of them).  The words have multipliers of their own: folded by a rotation
// they cancelled for values that repeat their low word in the high one, and all
// vectors of such a pool met in one slot.
template <int MM>
__device__ __forceinline__ uint32_t vec_hash(const int64_t (&y)[MM]) {
    uint32_t h = 0x243F6A88u;
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        h = (h ^ (uint32_t)y[k]) * 0x9E3779B1u + (uint32_t)((uint64_t)y[k] >> 32) * 0xC2B2AE3Du;
        h ^= h >> 15;
    }
    h *= 0x85EBCA77u;
    return h ^ (h >> 13);
}

// Open addressing in the global table of `mask + 1` slots (more than the row
// count, so a free slot always exists), linear probing from the vector's
// hash: a free slot (-1) is claimed with a compare-and-swap; a slot naming a
// row with the same vector takes min(that row, me) with an atomic minimum.
// Slots never change vector, so every row of a vector reaches the same slot,
// which ends holding the smallest row index offered for it.
template <int MM>
__device__ __forceinline__ void table_insert(const int64_t *__restrict__ obj, const int64_t (&y)[MM], uint32_t h,
                                             int32_t me, int32_t *__restrict__ table, uint32_t mask) {
    uint32_t s = h & mask;
    while (true) {
        int32_t q = table[s];
        if (q < 0) {
            q = atomicCAS(&table[s], -1, me);
            if (q < 0) return;  // claimed
        }
        bool eq = true;
#pragma unroll
        for (int k = 0; k < MM; ++k) eq &= obj[(int64_t)q * MM + k] == y[k];
        if (eq) {
            if (me < q) atomicMin(&table[s], me);
            return;
        }
        s = (s + 1) & mask;
    }
}

// Duplicate merging in two levels.  A sampler's pool repeats its most frequent
// cut vectors hundreds of thousands of times, and one global table slot per
// vector made those rows queue on a few cache lines.  So each block first
// merges a chunk of consecutive rows in an LDS table (the same probing, on the
// chunk's vectors staged in LDS, keeping the smallest row of the chunk per
// vector), and only the chunk's distinct vectors, with those rows, go to the
// global table.  The global minimum over the chunks' minima is the vector's
// smallest row.  Bound by latency, of the global inserts above all (a random
// slot, then a random row): the chunk's distinct vectors are listed first, so
// that one round of inserts, two at most, takes them all (a thread per eighth
// of the LDS slots took eight rounds, nearly empty ones).
constexpr int kDedupRows = 1008;   // rows per chunk: four blocks' LDS fit a CU at MM = 4
constexpr int kDedupSlots = 2048;  // LDS hash slots
constexpr int kDT = 512;           // threads per block: two rows each, 32 waves per CU

template <int MM>
__global__ __launch_bounds__(kDT) void dedupe_kernel(const int64_t *__restrict__ obj, int64_t M,
                                                    int32_t *__restrict__ table, uint32_t mask) {
    constexpr int SPT = kDedupSlots / kDT;  // slots per thread
    __shared__ __attribute__((aligned(16))) int64_t v[kDedupRows][MM];
    __shared__ int32_t loc[kDedupSlots];
    __shared__ int32_t have;
    for (int64_t c0 = (int64_t)blockIdx.x * kDedupRows; c0 < M; c0 += (int64_t)gridDim.x * kDedupRows) {
        const int len = (int)((M - c0) < kDedupRows ? (M - c0) : kDedupRows);
        for (int i = threadIdx.x; i < kDedupSlots; i += kDT) loc[i] = -1;
        if (threadIdx.x == 0) have = 0;
        for (int i = threadIdx.x; i < len * MM; i += kDT) (&v[0][0])[i] = obj[c0 * MM + i];
        __syncthreads();
        for (int p = threadIdx.x; p < len; p += kDT) {
            int64_t y[MM];
#pragma unroll
            for (int k = 0; k < MM; ++k) y[k] = v[p][k];
            uint32_t s = (vec_hash<MM>(y) >> 8) & (kDedupSlots - 1);
            while (true) {
                int32_t q = loc[s];
                if (q < 0) {
                    q = atomicCAS(&loc[s], -1, p);
                    if (q < 0) break;  // claimed
                }
                bool eq = true;
#pragma unroll
                for (int k = 0; k < MM; ++k) eq &= v[q][k] == y[k];
                if (eq) {
                    if (p < q) atomicMin(&loc[s], p);
                    break;
                }
                s = (s + 1) & (kDedupSlots - 1);
            }
        }
        __syncthreads();
        // the occupied slots, listed in the slots' own memory
        int32_t mine[SPT];
        int c = 0;
#pragma unroll
        for (int u = 0; u < SPT; ++u) {
            mine[u] = loc[u * kDT + threadIdx.x];
            c += mine[u] >= 0;
        }
        int at = c > 0 ? atomicAdd(&have, c) : 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SPT; ++u)
            if (mine[u] >= 0) loc[at++] = mine[u];
        __syncthreads();
        const int n = have;
        for (int i = threadIdx.x; i < n; i += kDT) {
            const int p = loc[i];
            int64_t y[MM];
#pragma unroll
            for (int k = 0; k < MM; ++k) y[k] = v[p][k];
            table_insert<MM>(obj, y, vec_hash<MM>(y), (int32_t)(c0 + p), table, mask);
        }
        __syncthreads();  // v, loc and have are rewritten for the next chunk
    }
}

// list[0 .. *count) = the rows named by the table's occupied slots, in no
// particular order.  Bound by reading the table; a block collects what it finds
// in LDS and takes one atomic per 4096 to 8192 rows (one per 4096 slots, all on
// the same word, took 50 us for 2^24 slots).
constexpr int kCollectBlocks = 512;
__global__ __launch_bounds__(kB) void collect_kernel(const int4 *__restrict__ table, int64_t quads,
                                                     int32_t *__restrict__ list, int64_t *__restrict__ count) {
    constexpr int kPer = 16 * kB;  // slots per step
    __shared__ int32_t buf[2 * kPer];
    __shared__ int32_t have;
    __shared__ int64_t base_sh;
    if (threadIdx.x == 0) have = 0;
    __syncthreads();
    auto flush = [&]() {
        const int nc = have;
        if (threadIdx.x == 0 && nc > 0) base_sh = (int64_t)atomicAdd((unsigned long long *)count, (unsigned long long)nc);
        __syncthreads();
        for (int i = threadIdx.x; i < nc; i += kB) list[base_sh + i] = buf[i];
        __syncthreads();
        if (threadIdx.x == 0) have = 0;
        __syncthreads();
    };
    const int64_t steps = (quads * 4 + kPer - 1) / kPer;
    for (int64_t st = blockIdx.x; st < steps; st += gridDim.x) {
        int32_t q[16];
        int c = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = st * (kPer / 4) + u * kB + threadIdx.x;
            const int4 v = i < quads ? table[i] : make_int4(-1, -1, -1, -1);
            q[4 * u] = v.x;
            q[4 * u + 1] = v.y;
            q[4 * u + 2] = v.z;
            q[4 * u + 3] = v.w;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) c += q[u] >= 0;
        if (c > 0) {
            int at = atomicAdd(&have, c);
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (q[u] >= 0) buf[at++] = q[u];
        }
        __syncthreads();
        const int full = have > kPer;
        __syncthreads();  // everybody has read `have` before the next step adds to it
        if (full) flush();
    }
    flush();
}

// The list that the pair pass compares: every distinct vector when there are
// at most kPairMax, else the rows left by pruning, or by the chunk pass when
// pruning left more than kPairMax.
struct PairList {
    const int32_t *all;      // distinct vectors, counts[0] of them
    const int32_t *pruned;   // left by pruning, counts[1] of them
    const int32_t *chunked;  // left by the chunk pass, counts[2] of them
    const int64_t *counts;
    __device__ __forceinline__ int route() const {
        return counts[0] <= kPairMax ? 0 : counts[1] <= kPairMax ? 1 : 2;
    }
    __device__ __forceinline__ const int32_t *list(int r) const { return r == 0 ? all : r == 1 ? pruned : chunked; }
};

// The bucket of a row in an ordered list, the largest keys first.  The key is a sum
// of the normalised values with falling weights (equal ones would put a front of
// constant sum into one bucket); every operation is monotone in floating point too,
// so a row's dominators lie in its bucket or an earlier one.
constexpr int kBuckets = 512;
template <int MM>
__device__ __forceinline__ int key_bucket(const int64_t (&y)[MM], const int64_t *__restrict__ lo,
                                          const int64_t *__restrict__ hi) {
    float key = 0.0f, w = 1.0f, top = 0.0f;
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        const double span = (double)hi[k] - (double)lo[k];
        const float scale = span > 0.0 ? (float)(1.0 / span) : 0.0f;
        key = fmaf(w, (float)(((double)y[k] - (double)lo[k]) * scale), key);
        top += w;
        w *= 0.70710678f;
    }
    return kBuckets - 1 - (int)fminf(fmaxf(key * ((float)kBuckets / top), 0.0f), (float)(kBuckets - 1));
}

// Chunk pass over a long pruned list, in any order: a row that another row of
// its chunk of 1024 dominates is dropped, the others are appended.  Each thread
// holds four rows in registers and walks the chunk once for all four (one
// broadcast LDS read of a row serves four comparisons), stopping when all four
// are dominated.  hist counts the rows left per bucket.
template <int MM>
__global__ __launch_bounds__(kB) void chunk_any_kernel(const int64_t *__restrict__ obj,
                                                       const int32_t *__restrict__ list, const int64_t *counts,
                                                       const int64_t *__restrict__ lo, const int64_t *__restrict__ hi,
                                                       int32_t *__restrict__ out, int64_t *out_count,
                                                       uint32_t *__restrict__ hist) {
    constexpr int RPT = kChunk / kB;  // rows per thread
    __shared__ int64_t v[kChunk][MM];
    const int64_t n = counts[1];
    if (counts[0] <= kPairMax || n <= kPairMax) return;
    for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < n; c0 += (int64_t)gridDim.x * kChunk) {
        const int len = (int)((n - c0) < kChunk ? (n - c0) : kChunk);
        for (int p = threadIdx.x; p < len; p += kB) {
            const int64_t *y = obj + (int64_t)list[c0 + p] * MM;
#pragma unroll
            for (int k = 0; k < MM; ++k) v[p][k] = y[k];
        }
        __syncthreads();
        int64_t y[RPT][MM];
        bool dom[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int j = r * kB + threadIdx.x;
            dom[r] = j >= len;
#pragma unroll
            for (int k = 0; k < MM; ++k) y[r][k] = j < len ? v[j][k] : 0;
        }
        for (int i = 0; i < len; ++i) {
            int64_t w[MM];
#pragma unroll
            for (int k = 0; k < MM; ++k) w[k] = v[i][k];
            bool done = true;
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                bool ge = i != r * kB + (int)threadIdx.x;
#pragma unroll
                for (int k = 0; k < MM; ++k) ge &= w[k] >= y[r][k];
                dom[r] |= ge;
                done &= dom[r];
            }
            if (done) break;
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int j = r * kB + threadIdx.x;
            const bool left = j < len && !dom[r];
            wave_append(left, left ? list[c0 + j] : 0, out, out_count);
            if (left) atomicAdd(&hist[key_bucket<MM>(y[r], lo, hi)], 1u);
        }
        __syncthreads();  // v is rewritten by the next chunk
    }
}

// fin[i] = the i-th listed row, packed[i] = its vector as 32-bit offsets from
// the first listed row's, dom[i] = 0; counts[3] = the list's length, counts[4]
// = 1 when some offset does not fit.  An ordered list (route 2): row i is the next
// one of its bucket (hist: rows per bucket, taken: rows placed so far), and
// limit[t] = where the bucket of tile t's last row ends.
template <int MM>
__global__ __launch_bounds__(kB) void pair_pack_kernel(const int64_t *__restrict__ obj, PairList L, int64_t *counts,
                                                       const int64_t *__restrict__ lo, const int64_t *__restrict__ hi,
                                                       const uint32_t *__restrict__ hist, uint32_t *__restrict__ taken,
                                                       int32_t *__restrict__ limit, int32_t *__restrict__ fin,
                                                       int32_t *__restrict__ packed, uint8_t *__restrict__ dom) {
    __shared__ uint32_t end[kBuckets], part[kB];
    const int route = L.route();
    const int64_t n = L.counts[route];
    if (blockIdx.x == 0 && threadIdx.x == 0) counts[3] = n;
    if (n == 0) return;
    if (route == 2) {  // inclusive sums of hist, two buckets per thread
        const uint32_t c0 = hist[2 * threadIdx.x], c1 = hist[2 * threadIdx.x + 1];
        part[threadIdx.x] = c0 + c1;
        __syncthreads();
        for (int off = 1; off < kB; off <<= 1) {
            const uint32_t o = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
            __syncthreads();
            part[threadIdx.x] += o;
            __syncthreads();
        }
        end[2 * threadIdx.x + 1] = part[threadIdx.x];
        end[2 * threadIdx.x] = part[threadIdx.x] - c1;
        __syncthreads();
    }
    int64_t base[MM];
    const int32_t *list = L.list(route);
    const int64_t r0 = list[0];
#pragma unroll
    for (int k = 0; k < MM; ++k) base[k] = obj[r0 * MM + k];
    bool wide = false;
    for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kB) {
        const int64_t r = list[i];
        int64_t y[MM];
#pragma unroll
        for (int k = 0; k < MM; ++k) y[k] = obj[r * MM + k];
        int64_t p = i;
        if (route == 2) {
            const int b = key_bucket<MM>(y, lo, hi);
            p = (int64_t)(b > 0 ? end[b - 1] : 0u) + atomicAdd(&taken[b], 1u);
            if (p % kB == kB - 1 || p == n - 1) limit[p / kB] = (int32_t)end[b];
        }
        fin[p] = (int32_t)r;
        dom[p] = 0;
#pragma unroll
        for (int k = 0; k < MM; ++k) {
            const uint64_t mag = y[k] >= base[k] ? (uint64_t)y[k] - (uint64_t)base[k] : (uint64_t)base[k] - (uint64_t)y[k];
            wide |= mag > 0x3fffffffull;  // differences of two offsets fit 32 bits
            packed[p * MM + k] = (int32_t)((uint64_t)y[k] - (uint64_t)base[k]);
        }
    }
    if (__ballot(wide) != 0 && (threadIdx.x & 63) == 0)
        atomicMax((unsigned long long *)&counts[4], 1ull);  // 1, whoever sets it
}

// Pair pass: dom[j] = 1 when some other listed vector is >= vector j
// componentwise.  ALU bound.  A work item is a tile of 256 rows j, one per
// lane, against up to 256 rows i; a wave reads row i through scalar loads
// (its address is uniform) and no LDS.  A pair takes MM subtractions with a
// scalar operand, whose signs are ORed over the objectives and ANDed over the
// rows i: MM + 2 vector instructions at MM = 4 (comparisons, each with its mask
// in a scalar register pair and a scalar AND, took 2.5 times as long).  Items run i tile by i tile, so that
// rows marked by the first tiles skip the later ones: a wave whose rows are all
// marked stops.  Concurrent marks all store the same byte.  The 64-bit form,
// for ranges past 32 bits, stages the rows i in LDS.
// An ordered list halves the pairs and puts the rows that dominate most first: a
// front of 600 000 points of two objectives 66 -> 39 ms, of eight with 64-bit
// differences 338 -> 108, 2 000 000 rows on forty nested fronts of eight 571 -> 182.
// hist and taken lie at the start of the bitmap of kept rows (cleared, if given).
template <int MM>
__global__ __launch_bounds__(kB) void pair_any_kernel(const int64_t *__restrict__ obj, const int64_t *__restrict__ counts,
                                                      const int32_t *__restrict__ limit, uint32_t *__restrict__ cleared,
                                                      const int32_t *__restrict__ fin,
                                                      const int32_t *__restrict__ packed, uint8_t *dom) {
    if (cleared != nullptr && blockIdx.x == 0)
        for (int i = threadIdx.x; i < 2 * kBuckets; i += kB) cleared[i] = 0u;
    const int64_t n = counts[3];
    const bool ordered = counts[0] > kPairMax && counts[1] > kPairMax;
    const bool wide = counts[4] != 0;
    const int64_t T = (n + kB - 1) / kB;
    // rows i per item: all 256, fewer where the list alone would not fill the
    // GPU (a chain of 256 rows is 11 us)
    const int isz = n > 8192 ? kB : n > 2048 ? 64 : 32;
    const int64_t TI = (n + isz - 1) / isz;
    __shared__ int64_t v[kB][MM];
    // item p = it * T + jt, stepped by the grid without a division per item
    const int64_t step_it = gridDim.x / std::max<int64_t>(T, 1), step_jt = gridDim.x - step_it * T;
    int64_t it = blockIdx.x / std::max<int64_t>(T, 1), jt = blockIdx.x - it * T;
    for (; it < TI; it += step_it, jt += step_jt) {
        if (jt >= T) {
            jt -= T;
            if (++it >= TI) break;
        }
        const int64_t i0 = it * isz;
        if (ordered && i0 >= limit[jt]) continue;
        const int64_t j = jt * kB + threadIdx.x;
        bool done = j >= n || dom[j] != 0;
        const int cnt = (int)((n - i0) < isz ? (n - i0) : isz);
        const bool diag = i0 / kB == jt;  // some rows i are rows j
        const int self = (int)(j - i0);
        bool hit = false;
        if (!wide) {
            if (__ballot(!done) == 0) continue;
            int32_t y[MM];
#pragma unroll
            for (int k = 0; k < MM; ++k) y[k] = j < n ? packed[j * MM + k] : 0;
            const int32_t *q = packed + i0 * MM;
            auto scan = [&](auto diagonal) __attribute__((always_inline)) {
                constexpr bool DIAG = decltype(diagonal)::value;
                int32_t miss = -1;  // sign bit set while every row has fallen short somewhere
                auto test = [&](int t) __attribute__((always_inline)) {
                    int32_t d = DIAG && t == self ? -1 : 0;
#pragma unroll
                    for (int k = 0; k < MM; ++k) d |= q[t * MM + k] - y[k];
                    miss &= d;
                };
                int t = 0;
                for (; t + 8 <= cnt; t += 8) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) test(t + u);
                    if (__ballot(!done && miss < 0) == 0) break;
                }
                if (t + 8 > cnt)
                    for (; t < cnt; ++t) test(t);
                hit = miss >= 0;
            };
            if (diag) scan(std::true_type{});
            else scan(std::false_type{});
        } else {
            if (!__syncthreads_or(done ? 0 : 1)) continue;
            if ((int)threadIdx.x < cnt) {
                const int64_t *y = obj + (int64_t)fin[i0 + threadIdx.x] * MM;
#pragma unroll
                for (int k = 0; k < MM; ++k) v[threadIdx.x][k] = y[k];
            }
            __syncthreads();
            if (!done) {
                const int64_t *y = obj + (int64_t)fin[j] * MM;
                int64_t yj[MM];
#pragma unroll
                for (int k = 0; k < MM; ++k) yj[k] = y[k];
                for (int t0 = 0; t0 < cnt && !hit; t0 += 4)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int t = min(t0 + u, cnt - 1);
                        bool ge = !diag || t != self;
#pragma unroll
                        for (int k = 0; k < MM; ++k) ge &= v[t][k] >= yj[k];
                        hit |= ge;
                    }
            }
            __syncthreads();  // v is rewritten by the next item
        }
        if (hit && !done) dom[j] = 1;
    }
}

// Ascending emission, pools of at most kEmitSmall rows: one block builds the
// bitmap of kept rows in LDS and writes the set bits in order.
constexpr int64_t kEmitSmall = 1 << 16;
__global__ __launch_bounds__(1024) void emit_small_kernel(const int32_t *__restrict__ fin,
                                                          const uint8_t *__restrict__ dom,
                                                          const int64_t *__restrict__ counts,
                                                          int64_t *__restrict__ keep, int64_t *__restrict__ num) {
    __shared__ uint32_t bits[kEmitSmall / 32];
    __shared__ int32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    bits[tid] = 0u;
    bits[tid + 1024] = 0u;
    __syncthreads();
    const int64_t n = counts[3];
    for (int64_t i = tid; i < n; i += 1024)
        if (dom[i] == 0) atomicOr(&bits[fin[i] >> 5], 1u << (fin[i] & 31));
    __syncthreads();
    const uint32_t w0 = bits[2 * tid], w1 = bits[2 * tid + 1];
    const int c = __popc(w0) + __popc(w1);
    int s = c;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(s, off);
        if (lane >= off) s += o;
    }
    if (lane == 63) wsum[wave] = s;
    __syncthreads();
    int64_t at = s - c;
    for (int w = 0; w < wave; ++w) at += wsum[w];
    for (uint64_t b = (uint64_t)w0 | ((uint64_t)w1 << 32); b; b &= b - 1)
        keep[at++] = (int64_t)tid * 64 + __ffsll((unsigned long long)b) - 1;
    if (tid == 1023) *num = at;
}

// Larger pools: the bitmap is in device memory (mark), a tile of 16384 rows (64 per
// thread) per block is counted, and each block adds up the tiles before its own
// (or reads their scanned sum, when there are many) and writes its set bits.
constexpr int64_t kEmitTile = 64 * kB;
constexpr int64_t kEmitScan = 4096;  // tiles past which the counts are scanned by a launch of their own

__global__ __launch_bounds__(kB) void mark_kernel(const int32_t *__restrict__ fin, const uint8_t *__restrict__ dom,
                                                  const int64_t *__restrict__ counts, uint32_t *__restrict__ bits) {
    const int64_t n = counts[3];
    for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kB)
        if (dom[i] == 0) atomicOr(&bits[fin[i] >> 5], 1u << (fin[i] & 31));
}

__device__ __forceinline__ int block_sum(int v, int *sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    int s = 0;
    for (int w = 0; w < kB / 64; ++w) s += sh[w];
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(kB) void emit_count_kernel(const uint64_t *__restrict__ bits, int64_t words,
                                                        uint32_t *__restrict__ cnt) {
    __shared__ int sh[kB / 64];
    const int64_t w = (int64_t)blockIdx.x * kB + threadIdx.x;
    const int s = block_sum(w < words ? __popcll(bits[w]) : 0, sh);
    if (threadIdx.x == 0) cnt[blockIdx.x] = (uint32_t)s;
}

// one block: exclusive scan of cnt[0 .. tiles) in place
__global__ __launch_bounds__(kB) void emit_scan_kernel(uint32_t *__restrict__ cnt, int64_t tiles) {
    __shared__ int sh[kB / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t c = 0; c < tiles; c += kB) {
        const int64_t i = c + threadIdx.x;
        const int v = i < tiles ? (int)cnt[i] : 0;
        int s = v;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(s, off);
            if (lane >= off) s += o;
        }
        if (lane == 63) sh[wave] = s;
        __syncthreads();
        int pre = 0, total = 0;
        for (int w = 0; w < kB / 64; ++w) {
            if (w < wave) pre += sh[w];
            total += sh[w];
        }
        if (i < tiles) cnt[i] = carry + (uint32_t)(pre + s - v);
        carry += (uint32_t)total;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kB) void emit_kernel(const uint64_t *__restrict__ bits, int64_t words,
                                                  const uint32_t *__restrict__ cnt, bool scanned,
                                                  int64_t *__restrict__ keep, int64_t *__restrict__ num) {
    __shared__ int sh[kB / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int before = 0;
    if (scanned) {
        before = (int)cnt[blockIdx.x];
    } else {
        for (int t = threadIdx.x; t < (int)blockIdx.x; t += kB) before += (int)cnt[t];
        before = block_sum(before, sh);
    }
    const int64_t w = (int64_t)blockIdx.x * kB + threadIdx.x;
    uint64_t b = w < words ? bits[w] : 0ull;
    const int c = __popcll(b);
    int s = c;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(s, off);
        if (lane >= off) s += o;
    }
    if (lane == 63) sh[wave] = s;
    __syncthreads();
    int64_t at = (int64_t)before + s - c;
    for (int q = 0; q < wave; ++q) at += sh[q];
    for (; b; b &= b - 1) keep[at++] = w * 64 + __ffsll((unsigned long long)b) - 1;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kB - 1) *num = at;
}

// Sort keys of objective k for the list of n = *d_n rows: key = hi_k - y_k
// (unsigned, exact), value = row.  The list is the survivors for the last
// objective, else the previous round's output (in A after an even number of
// digit passes, else in B).  Block 0 stores this round's digit-pass count.
__global__ void sort_key_kernel(const int64_t *__restrict__ obj, int m, int k, const int32_t *__restrict__ first,
                                const int64_t *__restrict__ d_n, const int64_t *__restrict__ lo,
                                const int64_t *__restrict__ hi, uint64_t *__restrict__ keyA, int32_t *valA,
                                const int32_t *valB, int32_t *__restrict__ passes) {
    const int64_t n = *d_n;
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    const uint64_t top = (uint64_t)hi[k];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint64_t span = n > 0 ? top - (uint64_t)lo[k] : 0;
        const int bits = span ? 64 - __clzll((long long)span) : 0;
        passes[k] = (bits + 7) / 8;
    }
    if (i >= n) return;
    const int32_t *src = k == m - 1 ? first : ((passes[k + 1] & 1) ? valB : valA);
    const int32_t r = src[i];
    keyA[i] = top - (uint64_t)obj[(int64_t)r * m + k];
    valA[i] = r;
}

// sorted[i] = the final round's output (objective 0's pass parity)
__global__ void settle_kernel(const int32_t *__restrict__ valA, const int32_t *__restrict__ valB,
                              const int32_t *__restrict__ passes, const int64_t *__restrict__ d_n,
                              int32_t *__restrict__ sorted) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < *d_n) sorted[i] = (passes[0] & 1) ? valB[i] : valA[i];
}

__global__ void unique_flag_kernel(const int64_t *__restrict__ obj, int m, const int32_t *__restrict__ idx,
                                   const int64_t *__restrict__ d_n, uint8_t *__restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= *d_n) return;
    uint8_t f = 1;
    if (i > 0) {
        const int64_t *a = obj + (int64_t)idx[i] * m, *b = obj + (int64_t)idx[i - 1] * m;
        f = 0;
        for (int k = 0; k < m; ++k) f |= a[k] != b[k];
    }
    flag[i] = f;
}

// Chunk pass over the list[0 .. U) of distinct vectors in lexicographic
// order: within each chunk of 1024, flag[p] = 0 when an earlier vector of the
// chunk is >= it componentwise.  Each thread holds four rows in registers and
// walks the chunk's earlier rows once for all four (one broadcast LDS read of
// a row serves four comparisons), stopping when all four are dominated.
template <int MM>
__global__ __launch_bounds__(kB) void chunk_nd_kernel(const int64_t *__restrict__ obj,
                                                      const int32_t *__restrict__ list,
                                                      const int64_t *__restrict__ d_U, uint8_t *__restrict__ flag) {
    constexpr int RPT = kChunk / kB;  // rows per thread
    __shared__ int64_t v[kChunk][MM];
    const int64_t U = *d_U;
    const int64_t c0 = (int64_t)blockIdx.x * kChunk;
    if (U <= kPairMax || c0 >= U) return;  // short lists take the pair pass
    const int len = (int)((U - c0) < kChunk ? (U - c0) : kChunk);
    for (int p = threadIdx.x; p < len; p += kB) {
        const int64_t *y = obj + (int64_t)list[c0 + p] * MM;
#pragma unroll
        for (int k = 0; k < MM; ++k) v[p][k] = y[k];
    }
    __syncthreads();
    int64_t y[RPT][MM];
    bool dom[RPT];
    int last = 0;  // rows before the thread's last live row
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int j = r * kB + threadIdx.x;
        dom[r] = j >= len;
        if (j < len) last = j;
#pragma unroll
        for (int k = 0; k < MM; ++k) y[r][k] = j < len ? v[j][k] : 0;
    }
    for (int i = 0; i < last; ++i) {
        int64_t w[MM];
#pragma unroll
        for (int k = 0; k < MM; ++k) w[k] = v[i][k];
        bool done = true;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            if (!dom[r] && i < r * kB + (int)threadIdx.x) {
                bool ge = true;
#pragma unroll
                for (int k = 0; k < MM; ++k) ge &= w[k] >= y[r][k];
                dom[r] = ge;
            }
            done &= dom[r];
        }
        if (done) break;
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int j = r * kB + threadIdx.x;
        if (j < len) flag[c0 + j] = dom[r] ? 0 : 1;
    }
}

// Survivor pass over sidx[0 .. S) (chunk survivors, lexicographic order): a
// survivor is kept when no earlier survivor is >= it componentwise.  Tiles of
// 256 earlier survivors pass through LDS; a block stops once all its rows are
// dominated.
template <int MM>
__global__ __launch_bounds__(kB) void global_nd_kernel(const int64_t *__restrict__ obj,
                                                       const int32_t *__restrict__ sidx,
                                                       const int64_t *__restrict__ d_U,
                                                       const int64_t *__restrict__ d_S,
                                                       uint8_t *__restrict__ keep) {
    __shared__ int64_t v[kB][MM];
    if (*d_U <= kPairMax) return;  // short lists take the pair pass
    const int64_t S = *d_S;
    const int64_t j0 = (int64_t)blockIdx.x * kB;
    if (j0 >= S) return;
    const int64_t j = j0 + threadIdx.x;
    const bool mine = j < S;
    int64_t yj[MM];
#pragma unroll
    for (int k = 0; k < MM; ++k) yj[k] = mine ? obj[(int64_t)sidx[j] * MM + k] : 0;
    bool alive = mine;
    for (int64_t i0 = 0; i0 < j0 + kB && i0 < S; i0 += kB) {
        const int64_t ii = i0 + threadIdx.x;
        if (ii < S) {
            const int64_t *y = obj + (int64_t)sidx[ii] * MM;
#pragma unroll
            for (int k = 0; k < MM; ++k) v[threadIdx.x][k] = y[k];
        }
        __syncthreads();
        if (alive) {
            const int lim = (int)((j - i0) < kB ? (j - i0) : kB);  // earlier survivors only
            for (int t = 0; t < lim; ++t) {
                bool ge = true;
#pragma unroll
                for (int k = 0; k < MM; ++k) ge &= v[t][k] >= yj[k];
                if (ge) {
                    alive = false;
                    break;
                }
            }
        }
        if (!__syncthreads_or(alive ? 1 : 0)) break;
    }
    if (alive) keep[sidx[j]] = 1;
}

// Pair pass of the ranks for lists of at most kPairMax vectors: the chunk and
// survivor passes above leave most
// CUs idle on a few thousand rows (one block per chunk, one per 256
// survivors, each walking its earlier rows in sequence), so short lists are
// instead split into 256-row tiles and every tile pair (it, jt) with
// it <= jt is one work item of a persistent grid.  Row j of tile jt is marked
// (dom[j] = 1) when a row i < j of tile it is >= it componentwise: in the
// lexicographic order every dominator comes first, and the vectors are
// distinct, so "some earlier row is >= it" is exactly "dominated".  A row
// already marked by another pair skips its comparisons, and a pair whose rows
// are all marked is skipped; concurrent marks all store the same byte.
template <int MM>
__global__ __launch_bounds__(kB) void pair_nd_kernel(const int64_t *__restrict__ obj,
                                                     const int32_t *__restrict__ list,
                                                     const int64_t *__restrict__ d_n, uint8_t *dom) {
    const int64_t n = *d_n;
    if (n > kPairMax) return;
    const int T = (int)((n + kB - 1) / kB);
    const int P = T * (T + 1) / 2;
    __shared__ int64_t v[kB][MM];
    for (int p = blockIdx.x; p < P; p += gridDim.x) {
        // p = jt (jt + 1) / 2 + it, 0 <= it <= jt
        int jt = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);
        while (jt * (jt + 1) / 2 > p) --jt;
        while ((jt + 1) * (jt + 2) / 2 <= p) ++jt;
        const int it = p - jt * (jt + 1) / 2;
        const int64_t j = (int64_t)jt * kB + threadIdx.x;
        const bool live = j < n && dom[j] == 0;
        if (!__syncthreads_or(live ? 1 : 0)) continue;
        const int64_t i = (int64_t)it * kB + threadIdx.x;
        if (i < n) {
            const int64_t *y = obj + (int64_t)list[i] * MM;
#pragma unroll
            for (int k = 0; k < MM; ++k) v[threadIdx.x][k] = y[k];
        }
        __syncthreads();
        if (live) {
            int64_t yj[MM];
            const int64_t *y = obj + (int64_t)list[j] * MM;
#pragma unroll
            for (int k = 0; k < MM; ++k) yj[k] = y[k];
            // tile it < jt is full (only the last tile can be partial)
            const int lim = it < jt ? kB : (int)threadIdx.x;
            for (int t = 0; t < lim; ++t) {
                bool ge = true;
#pragma unroll
                for (int k = 0; k < MM; ++k) ge &= v[t][k] >= yj[k];
                if (ge) {
                    dom[j] = 1;
                    break;
                }
            }
        }
        __syncthreads();  // v is rewritten by the next pair
    }
}

// keep[list[j]] = 1 for the unmarked rows of a short list.
__global__ __launch_bounds__(kB) void pair_keep_kernel(const int32_t *__restrict__ list,
                                                       const int64_t *__restrict__ d_n,
                                                       const uint8_t *__restrict__ dom, uint8_t *__restrict__ keep) {
    const int64_t n = *d_n;
    const int64_t j = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (n <= kPairMax && j < n && dom[j] == 0) keep[list[j]] = 1;
}

// Both routes are queued; the list length, known only on the device, picks
// the one that works (the other's launches return at once).
template <int MM>
void launch_nd_passes(const int64_t *obj, const int32_t *list, const int64_t *d_n, int64_t cap, uint8_t *flag,
                      int32_t *sidx, int64_t *d_s, uint32_t *cnt, uint8_t *keep, hipStream_t st) {
    const int64_t short_cap = std::min<int64_t>(cap, kPairMax);
    const int64_t tc = (short_cap + kB - 1) / kB;
    hipLaunchKernelGGL(fill_u8_kernel, dim3(grid_for_n(short_cap, kB)), dim3(kB), 0, st, flag, short_cap, (uint8_t)0);
    hipLaunchKernelGGL(pair_nd_kernel<MM>, dim3((unsigned)std::max<int64_t>(std::min<int64_t>(tc * (tc + 1) / 2, kPairBlocks), 1)),
                       dim3(kB), 0, st, obj, list, d_n, flag);
    hipLaunchKernelGGL(pair_keep_kernel, dim3(grid_for_n(short_cap, kB)), dim3(kB), 0, st, list, d_n, flag, keep);
    QAIA_HIP(hipGetLastError());
    if (cap <= kPairMax) return;
    hipLaunchKernelGGL(chunk_nd_kernel<MM>, dim3(grid_for_n(cap, kChunk)), dim3(kB), 0, st, obj, list, d_n, flag);
    QAIA_HIP(hipGetLastError());
    select_flagged<int32_t, int32_t>(list, flag, d_n, cap, sidx, d_s, cnt, nullptr, st);
    hipLaunchKernelGGL(global_nd_kernel<MM>, dim3(grid_for_n(cap, kB)), dim3(kB), 0, st, obj, sidx, d_n, d_s, keep);
    QAIA_HIP(hipGetLastError());
}

// The non-dominated rows of the lexicographically ordered distinct vectors
// list[0 .. n) (n = *d_n <= cap): keep[row] = 1 (keep is not cleared here).
// sidx / d_s receive the chunk survivors.
void nd_passes(const int64_t *obj, int32_t m, const int32_t *list, const int64_t *d_n, int64_t cap, uint8_t *flag,
               int32_t *sidx, int64_t *d_s, uint32_t *cnt, uint8_t *keep, hipStream_t st) {
    switch (m) {
#define QAIA_ND(MM) \
    case MM: launch_nd_passes<MM>(obj, list, d_n, cap, flag, sidx, d_s, cnt, keep, st); break;
        QAIA_ND(1)
        QAIA_ND(2)
        QAIA_ND(3)
        QAIA_ND(4)
        QAIA_ND(5)
        QAIA_ND(6)
        QAIA_ND(7)
        QAIA_ND(8)
#undef QAIA_ND
        default: throw Error{QAIA_UNSUPPORTED, "the filter supports 1..8 objectives"};
    }
}

// ranks: rows of the current list that entered rank r leave the list
__global__ void rank_assign_kernel(const int32_t *__restrict__ list, const int64_t *__restrict__ d_n,
                                   uint8_t *__restrict__ keep, int32_t r, int32_t *__restrict__ rank,
                                   uint8_t *__restrict__ rem) {
    const int64_t p = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (p >= *d_n) return;
    const int32_t s = list[p];
    const bool in_front = keep[s] != 0;
    if (in_front) {
        rank[s] = r;
        keep[s] = 0;
    }
    rem[p] = in_front ? 0 : 1;
}

__global__ void rank_fill_kernel(const int32_t *__restrict__ list, int64_t n, int32_t r, int32_t *__restrict__ rank) {
    const int64_t p = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (p < n) rank[list[p]] = r;
}

// every sorted position takes the rank of its run's representative
__global__ void rank_spread_kernel(const int32_t *__restrict__ sorted, const int32_t *__restrict__ run,
                                   const int32_t *__restrict__ uidx, int64_t M, int32_t *__restrict__ rank) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= M) return;
    const int32_t rep = uidx[run[i] - 1];
    const int32_t s = sorted[i];
    if (s != rep) rank[s] = rank[rep];
}



// Per-objective minimum over the rows of a pool (the reference point of the
// hypervolume comparisons in section "Comparison to evolutionary
// algorithm-based heuristics" is the worst value of each objective).  The pool is
// read as a flat array by a multiple of m threads, so that a thread stays with
// one objective and a wave's loads are contiguous; the block merges in LDS, and one
// atomic min per objective and block merges the blocks.  Those are serial at some
// 10 ns each, hence few large blocks: 570 000 rows of three objectives 28 us with
// rows per thread and 2048 blocks, now 6.3 (1024 threads, 256 blocks).
__global__ void objective_min_init_kernel(int64_t *lo, int m) {
    if ((int)threadIdx.x < m) lo[threadIdx.x] = INT64_MAX;
}

constexpr int kMinThreads = 1024, kMinBlocks = 256;

__global__ __launch_bounds__(kMinThreads) void objective_min_kernel(const int64_t *__restrict__ obj, int64_t M, int m,
                                                                    int64_t *__restrict__ lo) {
    __shared__ long long red[8];
    if (threadIdx.x < 8) red[threadIdx.x] = INT64_MAX;
    __syncthreads();
    const int threads = (int)(gridDim.x * kMinThreads) / m * m;  // at most 2^18
    const int t = (int)(blockIdx.x * kMinThreads + threadIdx.x);
    if (t < threads) {
        int64_t mn = INT64_MAX;
#pragma unroll 4
        for (int64_t i = t; i < M * m; i += threads) mn = min(mn, obj[i]);
        atomicMin(&red[t % m], (long long)mn);
    }
    __syncthreads();
    if ((int)threadIdx.x < m) atomicMin((long long *)&lo[threadIdx.x], red[threadIdx.x]);
}


// Workspace of the ranks.  The first 64 bytes hold the device counts: [0]
// unique vectors, [1] chunk survivors, [2] rows.
struct PLayout {
    size_t counts = 0, passes, lo, hi;
    size_t flag, keep, surv, keyA, keyB, valA, valB, sorted, uidx, sidx, hist, total, cnt;
    size_t list2, rem, run;
    size_t total_bytes = 0;
};

PLayout layout(int64_t M) {
    PLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align256(bytes);
        return o;
    };
    const size_t Mz = (size_t)std::max<int64_t>(M, 1);
    L.counts = take(8 * 8);
    L.passes = take(4 * 8);
    L.lo = take(8 * 8);
    L.hi = take(8 * 8);
    L.flag = take(Mz);
    L.keep = take(Mz);
    L.surv = take(4 * Mz);
    L.keyA = take(8 * Mz);
    L.keyB = take(8 * Mz);
    L.valA = take(4 * Mz);
    L.valB = take(4 * Mz);
    L.sorted = take(4 * Mz);
    L.uidx = take(4 * Mz);
    L.sidx = take(4 * Mz);
    L.hist = take(4 * radix_hist_words(M));
    L.total = take(4 * 256);
    L.cnt = take(4 * select_cnt_words(M));
    L.list2 = take(4 * Mz);
    L.rem = take(Mz);
    L.run = take(4 * Mz);
    L.total_bytes = off;
    return L;
}

// Workspace of the filter.  Counts: [0] distinct vectors, [1] left by pruning,
// [2] left by the chunk pass, [3] the pair pass's list, [4] wide range.
struct FLayout {
    size_t counts = 0, lo, hi, best, bits, cnt, all, pruned, fin, dom, packed, table;
    int64_t words = 0;  // 64-bit words of the bitmap
    uint64_t table_slots = 0;
    size_t total_bytes = 0;
};

FLayout filter_layout(int64_t M, int32_t m) {
    FLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align256(bytes);
        return o;
    };
    const size_t Mz = (size_t)std::max<int64_t>(M, 1);
    L.words = (int64_t)(Mz + 63) / 64;
    L.counts = take(8 * 8);
    L.lo = take(8 * 8);
    L.hi = take(8 * 8);
    L.best = take(8 * kDirs);
    L.bits = take(8 * (size_t)L.words);
    L.cnt = take(4 * (((size_t)Mz + kEmitTile - 1) / kEmitTile));
    L.all = take(4 * Mz);
    L.pruned = take(4 * Mz);
    L.fin = take(4 * Mz);
    L.dom = take(Mz);
    // a power of two of at least 1.5 M slots (load factor <= 2/3)
    uint64_t c = 1024;
    while (c < (uint64_t)Mz + Mz / 2) c <<= 1;
    L.table_slots = c;
    // the offsets are written once the table's slots have been collected
    L.table = L.packed = take(std::max<size_t>(4 * c, 4 * Mz * (size_t)std::min(std::max(m, 1), 8)));
    L.total_bytes = off;
    return L;
}

unsigned grid_for(int64_t n, int per = kB) {
    int64_t g = (n + per - 1) / per;
    return (unsigned)std::max<int64_t>(g, 1);
}

struct PView {
    int64_t *counts, *lo, *hi;
    int32_t *passes, *surv, *valA, *valB, *sorted, *uidx, *sidx;
    uint8_t *flag, *keep;
    uint64_t *keyA, *keyB;
    uint32_t *hist, *total, *cnt;
};

PView view(void *ws, const PLayout &L) {
    char *b = (char *)ws;
    PView v;
    v.counts = (int64_t *)(b + L.counts);
    v.passes = (int32_t *)(b + L.passes);
    v.lo = (int64_t *)(b + L.lo);
    v.hi = (int64_t *)(b + L.hi);
    v.surv = (int32_t *)(b + L.surv);
    v.valA = (int32_t *)(b + L.valA);
    v.valB = (int32_t *)(b + L.valB);
    v.sorted = (int32_t *)(b + L.sorted);
    v.uidx = (int32_t *)(b + L.uidx);
    v.sidx = (int32_t *)(b + L.sidx);
    v.flag = (uint8_t *)(b + L.flag);
    v.keep = (uint8_t *)(b + L.keep);
    v.keyA = (uint64_t *)(b + L.keyA);
    v.keyB = (uint64_t *)(b + L.keyB);
    v.hist = (uint32_t *)(b + L.hist);
    v.total = (uint32_t *)(b + L.total);
    v.cnt = (uint32_t *)(b + L.cnt);
    return v;
}

// list[i] = i and *count = n
__global__ void iota_kernel(int32_t *__restrict__ list, int64_t n, int64_t *__restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i == 0) *count = n;
    if (i < n) list[i] = (int32_t)i;
}

template <int MM>
void launch_range(const int64_t *obj, int64_t M, const PView &v, hipStream_t st) {
    hipLaunchKernelGGL(range_init_kernel, dim3(1), dim3(64), 0, st, v.lo, v.hi, MM);
    hipLaunchKernelGGL((sample_range_kernel<MM, false>), dim3((unsigned)std::min<int64_t>(grid_for(M), 4096)), dim3(kB),
                       0, st, obj, RowList{nullptr, nullptr, M}, v.lo, v.hi);
}

// Sort all M rows lexicographically descending (ties by index): v.sorted[0 ..
// M), counts[2] = M.
void sort_rows(const int64_t *obj, int64_t M, int32_t m, const PView &v, hipStream_t st) {
    switch (m) {
#define QAIA_RANGE(MM) \
    case MM: launch_range<MM>(obj, M, v, st); break;
        QAIA_RANGE(1)
        QAIA_RANGE(2)
        QAIA_RANGE(3)
        QAIA_RANGE(4)
        QAIA_RANGE(5)
        QAIA_RANGE(6)
        QAIA_RANGE(7)
        QAIA_RANGE(8)
#undef QAIA_RANGE
        default: throw Error{QAIA_UNSUPPORTED, "the filter supports 1..8 objectives"};
    }
    int64_t *d_S = v.counts + 2;
    hipLaunchKernelGGL(iota_kernel, dim3(grid_for(M)), dim3(kB), 0, st, v.surv, M, d_S);
    QAIA_HIP(hipGetLastError());
    for (int k = m - 1; k >= 0; --k) {
        hipLaunchKernelGGL(sort_key_kernel, dim3(grid_for(M)), dim3(kB), 0, st, obj, m, k, v.surv, d_S, v.lo, v.hi,
                           v.keyA, v.valA, v.valB, v.passes);
        QAIA_HIP(hipGetLastError());
        for (int pass = 0; pass < 8; ++pass) {
            const bool even = (pass & 1) == 0;
            radix_pass(even ? v.keyA : v.keyB, even ? v.valA : v.valB, even ? v.keyB : v.keyA,
                       even ? v.valB : v.valA, M, d_S, v.passes + k, pass, v.hist, v.total, st);
        }
    }
    hipLaunchKernelGGL(settle_kernel, dim3(grid_for(M)), dim3(kB), 0, st, v.valA, v.valB, v.passes, d_S, v.sorted);
    QAIA_HIP(hipGetLastError());
}

template <int MM>
void launch_filter(const int64_t *obj, int64_t M, int64_t *keep_idx, int64_t *num_keep, char *b, const FLayout &L,
                   hipStream_t st) {
    int64_t *counts = (int64_t *)(b + L.counts), *lo = (int64_t *)(b + L.lo), *hi = (int64_t *)(b + L.hi);
    unsigned long long *best = (unsigned long long *)(b + L.best);
    uint64_t *bits = (uint64_t *)(b + L.bits);
    uint32_t *cnt = (uint32_t *)(b + L.cnt);
    int32_t *all = (int32_t *)(b + L.all);
    int32_t *table = (int32_t *)(b + L.table), *pruned = (int32_t *)(b + L.pruned), *fin = (int32_t *)(b + L.fin);
    int32_t *packed = (int32_t *)(b + L.packed);
    uint8_t *dom = (uint8_t *)(b + L.dom);
    const bool small = M <= kEmitSmall;
    hipLaunchKernelGGL(filter_init_kernel, dim3((unsigned)std::min<int64_t>(grid_for((int64_t)L.table_slots / 4), 2048)),
                       dim3(kB), 0, st, (int4 *)table, (int64_t)L.table_slots / 4, (uint32_t *)bits,
                       M > kPairMax ? 2 * L.words : 0, counts, best, lo, hi);
    hipLaunchKernelGGL(dedupe_kernel<MM>, dim3((unsigned)std::min<int64_t>(grid_for(M, kDedupRows), 4096)), dim3(kDT),
                       0, st, obj, M, table, (uint32_t)(L.table_slots - 1));
    hipLaunchKernelGGL(collect_kernel, dim3((unsigned)std::min<int64_t>(grid_for((int64_t)L.table_slots, 16 * kB), kCollectBlocks)),
                       dim3(kB), 0, st, (const int4 *)table, (int64_t)L.table_slots / 4, all, counts + 0);
    QAIA_HIP(hipGetLastError());
    const RowList distinct{all, counts + 0, 0};
    // the chunk survivors reuse the distinct list's memory: by then only the pruned list is read
    int32_t *chunked = all;
    // an ordered list's counters take the start of the bitmap, which the marks need later; its limits
    // the pruned list's memory
    uint32_t *hist = M > kPairMax ? (uint32_t *)bits : nullptr;
    static_assert(kPairMax / 8 >= 8 * kBuckets, "both counters fit the bitmap of more than kPairMax rows");
    int32_t *limit = pruned;
    if (M > kPairMax) {
        const int64_t sample = std::min<int64_t>(M, kSampleRows);
        hipLaunchKernelGGL((sample_range_kernel<MM, true>), dim3((unsigned)std::min<int64_t>(grid_for(sample), 512)),
                           dim3(kB), 0, st, obj, distinct, lo, hi);
        hipLaunchKernelGGL(pivot_cand_kernel<MM>, dim3((unsigned)std::min<int64_t>(grid_for(sample), kCandBlocks)),
                           dim3(kB), 0, st, obj, distinct, lo, hi, best);
        hipLaunchKernelGGL(prune_kernel<MM>, dim3((unsigned)std::min<int64_t>(grid_for(M, 64), 2048)), dim3(kB), 0, st,
                           obj, distinct, best, pruned, counts + 1);
        hipLaunchKernelGGL(chunk_any_kernel<MM>, dim3((unsigned)std::min<int64_t>(grid_for(M, kChunk), 4096)), dim3(kB),
                           0, st, obj, pruned, counts, lo, hi, chunked, counts + 2, hist);
    }
    hipLaunchKernelGGL(pair_pack_kernel<MM>, dim3((unsigned)std::min<int64_t>(grid_for(M), 1024)), dim3(kB), 0, st, obj,
                       PairList{all, pruned, chunked, counts}, counts, lo, hi, hist,
                       hist ? hist + kBuckets : nullptr, limit, fin, packed, dom);
    const int64_t tiles = grid_for(M);
    hipLaunchKernelGGL(pair_any_kernel<MM>, dim3((unsigned)std::min<int64_t>(tiles * tiles * 8, kPairBlocks)), dim3(kB), 0,
                       st, obj, counts, limit, hist, fin, packed, dom);
    if (small) {
        hipLaunchKernelGGL(emit_small_kernel, dim3(1), dim3(1024), 0, st, fin, dom, counts, keep_idx, num_keep);
    } else {
        const int64_t etiles = (M + kEmitTile - 1) / kEmitTile;
        const bool scan = etiles > kEmitScan;
        hipLaunchKernelGGL(mark_kernel, dim3((unsigned)std::min<int64_t>(grid_for(M), 1024)), dim3(kB), 0, st, fin, dom,
                           counts, (uint32_t *)bits);
        hipLaunchKernelGGL(emit_count_kernel, dim3((unsigned)etiles), dim3(kB), 0, st, bits, L.words, cnt);
        if (scan) hipLaunchKernelGGL(emit_scan_kernel, dim3(1), dim3(kB), 0, st, cnt, etiles);
        hipLaunchKernelGGL(emit_kernel, dim3((unsigned)etiles), dim3(kB), 0, st, bits, L.words, cnt, scan, keep_idx,
                           num_keep);
    }
    QAIA_HIP(hipGetLastError());
}

}  // namespace

size_t pareto_ws_bytes(int64_t M, int32_t m) { return filter_layout(M, m).total_bytes; }

void launch_pareto(const int64_t *obj, int64_t M, int32_t m, int64_t *keep_idx, int64_t *num_keep,
                   void *ws, size_t ws_bytes, hipStream_t st) {
    if (M == 0) {
        hipLaunchKernelGGL(fill_i64_kernel, dim3(1), dim3(kB), 0, st, num_keep, (int64_t)1, (int64_t)0);
        QAIA_HIP(hipGetLastError());
        return;
    }
    const FLayout L = filter_layout(M, m);
    QAIA_CHECK(ws_bytes >= L.total_bytes, QAIA_WORKSPACE_TOO_SMALL,
               "pareto filter workspace needs " + std::to_string(L.total_bytes) + " bytes");
    switch (m) {
#define QAIA_FILTER(MM) \
    case MM: launch_filter<MM>(obj, M, keep_idx, num_keep, (char *)ws, L, st); break;
        QAIA_FILTER(1)
        QAIA_FILTER(2)
        QAIA_FILTER(3)
        QAIA_FILTER(4)
        QAIA_FILTER(5)
        QAIA_FILTER(6)
        QAIA_FILTER(7)
        QAIA_FILTER(8)
#undef QAIA_FILTER
        default: throw Error{QAIA_UNSUPPORTED, "the filter supports 1..8 objectives"};
    }
}

void launch_objective_min(const int64_t *obj, int64_t M, int32_t m, int64_t *lo, bool accumulate,
                          hipStream_t st) {
    if (!accumulate) hipLaunchKernelGGL(objective_min_init_kernel, dim3(1), dim3(64), 0, st, lo, m);
    if (M > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>((M * m + kMinThreads - 1) / kMinThreads, kMinBlocks);
        hipLaunchKernelGGL(objective_min_kernel, dim3(grid), dim3(kMinThreads), 0, st, obj, M, m, lo);
    }
    QAIA_HIP(hipGetLastError());
}

size_t pareto_ranks_ws_bytes(int64_t M, int32_t m) {
    (void)m;
    return layout(M).total_bytes;
}

// Non-dominated sorting by peeling: sort and de-duplicate as the filter does
// (without pruning: every row needs a rank), then repeatedly take the
// non-dominated set of the remaining unique vectors (chunk pass + survivor
// pass, as above) as the next rank and remove it; the list stays in
// lexicographic order, a linear extension of dominance, which the two passes
// rely on.  Duplicates take their representative's rank.
int32_t launch_pareto_ranks(const int64_t *obj, int64_t M, int32_t m, int32_t max_rank, int32_t *rank, void *ws,
                            size_t ws_bytes, hipStream_t st) {
    if (M == 0) return 0;
    const PLayout L = layout(M);
    QAIA_CHECK(ws_bytes >= L.total_bytes, QAIA_WORKSPACE_TOO_SMALL,
               "pareto ranks workspace needs " + std::to_string(L.total_bytes) + " bytes");
    QAIA_CHECK(M <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many rows");
    char *b = (char *)ws;
    const PView v = view(ws, L);
    uint8_t *rem = (uint8_t *)(b + L.rem);
    int32_t *list2 = (int32_t *)(b + L.list2), *run = (int32_t *)(b + L.run);
    hipLaunchKernelGGL(fill_u8_kernel, dim3(grid_for(M)), dim3(kB), 0, st, v.keep, M, (uint8_t)0);
    QAIA_HIP(hipGetLastError());
    sort_rows(obj, M, m, v, st);
    int32_t *cur = v.sorted;
    const int64_t *d_M = v.counts + 2;
    hipLaunchKernelGGL(unique_flag_kernel, dim3(grid_for(M)), dim3(kB), 0, st, obj, m, cur, d_M, v.flag);
    QAIA_HIP(hipGetLastError());
    // uidx: the representatives; run[i]: 1 + index of position i's run
    select_flagged<int32_t, int32_t>(cur, v.flag, d_M, M, v.uidx, v.counts + 0, v.cnt, run, st);
    // the working list starts as the unique representatives (a copy, uidx is kept for the spread)
    int32_t *list = v.surv, *other = list2;
    QAIA_HIP(hipMemcpyAsync(list, v.uidx, sizeof(int32_t) * (size_t)M, hipMemcpyDeviceToDevice, st));
    int64_t n = 0;
    QAIA_HIP(hipMemcpyAsync(&n, v.counts + 0, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    QAIA_HIP(hipStreamSynchronize(st));
    int32_t r = 0;
    while (n > 0) {
        if (r == max_rank) {
            hipLaunchKernelGGL(rank_fill_kernel, dim3(grid_for(n)), dim3(kB), 0, st, list, n, r, rank);
            QAIA_HIP(hipGetLastError());
            break;
        }
        // the list length n (= counts[0]) is also known on the host here
        nd_passes(obj, m, list, v.counts + 0, n, v.flag, v.sidx, v.counts + 1, v.cnt, v.keep, st);
        hipLaunchKernelGGL(rank_assign_kernel, dim3(grid_for(n)), dim3(kB), 0, st, list, v.counts + 0, v.keep, r, rank,
                           rem);
        QAIA_HIP(hipGetLastError());
        select_flagged<int32_t, int32_t>(list, rem, nullptr, n, other, v.counts + 0, v.cnt, nullptr, st);
        std::swap(list, other);
        QAIA_HIP(hipMemcpyAsync(&n, v.counts + 0, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        QAIA_HIP(hipStreamSynchronize(st));
        ++r;
    }
    hipLaunchKernelGGL(rank_spread_kernel, dim3(grid_for(M)), dim3(kB), 0, st, cur, run, v.uidx, M, rank);
    QAIA_HIP(hipGetLastError());
    return r;
}

}  // namespace qaia
