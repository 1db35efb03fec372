// Launches of the one-spin-per-lane sparse kernel (group.hpp): shapes, the rule
// that picks one, and the four-replica instantiations.
#include <algorithm>
#include <numeric>

#include "group.hpp"

namespace qaia {

// lane order (falling degree) and each node's place in it
void group_order(const Problem &p, std::vector<int32_t> &order, std::vector<int32_t> &place) {
    order.resize(p.n);
    place.resize(p.n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return p.rowptr[a + 1] - p.rowptr[a] > p.rowptr[b + 1] - p.rowptr[b];
    });
    for (int i = 0; i < p.n; ++i) place[order[i]] = i;
}

namespace {

struct GroupShape { int nt, npt; };
// lanes per block (at most) x spins per lane
constexpr GroupShape kGroupShapes[7] = {{64, 1}, {64, 2}, {64, 4}, {256, 2}, {256, 4}, {512, 1}, {512, 2}};
// Four replicas per lane from this many spin-lanes (rows x n) on: 42 spins x
// 16 000 replicas 479 -> 357 us per 1000 steps, x 3200 179 -> 254; 512 spins x 1024
// replicas 0.69 -> 0.54 us per step.
constexpr int64_t kFourMin = (int64_t)8 * 64 * 1024;
// One spin per lane and up to eight waves per group below this many lanes (per
// replicas held): 200 spins x 1024 replicas 0.58 -> 0.35 us per step at V = 1, x
// 4096 0.81 -> 0.92; 512 spins x 1024 replicas 0.67 -> 0.54 at V = 4, x 4096 1.00 ->
// 1.15.
constexpr int64_t kWideMax1 = (int64_t)10 * 64 * 1024, kWideMax4 = (int64_t)20 * 64 * 1024;

// One wave per group where the spins fit (no barrier); else, where the GPU is
// full, several spins per lane (fewer waves to wait for each other: n = 512,
// 32 768 replicas, V = 4: 5.9 us per step with 256 lanes, 7.1 with 512), and where
// it is not, or where neighbour lists of more than eight take the registers, one
// spin per lane (n = 512, 80 replicas: 0.29 against 0.37 us per step; n = 300,
// degree up to 19, 32 768 replicas: 16 against 25).  With noise or tracing, which the
// draws bind and which need whole groups side by side, several spins per lane
// throughout (noise, 32 768 replicas, against the tiled kernel: n = 512, mean degree
// 15, 301 -> 91 us per step; n = 1000, mean degree 12, 1091 -> 404, one wave per SIMD).
int group_shape(int n, int maxdeg, int V, bool full, int64_t lanes) {
    if (n <= 64) return 0;
    if (n <= 128) return 1;
    if (full) return n <= 512 ? 3 : 4;
    const bool wide = V == 1 ? lanes < kWideMax1 || maxdeg > 8 : lanes < kWideMax4 || maxdeg > 8;
    if (wide) return n <= 512 ? 5 : 6;
    return n <= 256 ? 2 : n <= 512 ? 3 : 4;
}

}  // namespace

bool sparse_group_fits(const Problem &p) {
    return p.n <= 1024 && p.max_degree <= 32 && p.m <= 8;
}

void launch_sparse_group(const Problem &p, int64_t W, int32_t R, const qaia_schedule &s, void *ws, const WsLayout &L,
                         uint64_t *spins, int64_t *obj, float *trace, int32_t trace_steps, hipStream_t st) {
    const int64_t rows = W * (int64_t)R;
    if (rows == 0) return;
    char *b = (char *)ws;
    GroupArgs a{};
    a.n = p.n;
    a.m = p.m;
    a.words = p.words;
    a.R = R;
    a.T = s.steps;
    a.E = p.E;
    a.order = p.d_order;
    a.place = p.d_place;
    a.rowptr = p.d_rowptr;
    a.col = p.d_col;
    a.eid = p.d_eid;
    a.Wt = p.d_W;
    a.eu = p.d_eu;
    a.ev = p.d_ev;
    a.jcp = (const float *)(b + L.jcp);
    a.c0s = (const double *)(b + L.c0s);
    a.kt_tab = (const float *)(b + L.kt);
    a.dta0 = s.dt * s.a0;
    a.dt_alpha = s.dt * s.noise_alpha;
    a.amp = s.init_amp;
    a.seed = s.seed;
    a.offset = s.replica_offset;
    a.spins = spins;
    a.obj = obj;
    a.trace = trace;
    a.trace_steps = trace_steps;
    const bool dsb = s.variant == QAIA_DSB, full = a.dt_alpha != 0.0f || trace != nullptr;
    const int n = p.n;
    const int64_t lanes = rows * n;  // spin-per-lane work at V = 1
    const int V = !full && R >= 4 && lanes >= kFourMin ? 4 : 1;
    const int shape = group_shape(n, p.max_degree, V, full, lanes);
    const GroupShape gs = kGroupShapes[shape];
    int NT = std::max(64, (n + gs.npt * 64 - 1) / (gs.npt * 64) * 64);
    if (full && gs.nt > 64) NT = gs.nt;  // noise is ALU bound: whole groups side by side fill the lanes
    a.groups_per_w = (R + V - 1) / V;
    a.groups = W * a.groups_per_w;
    a.per_block = NT * gs.npt / n;
    const int64_t blocks = (a.groups + a.per_block - 1) / a.per_block;
    QAIA_CHECK(blocks <= INT32_MAX, QAIA_INVALID_ARGUMENT, "too many replicas for one launch");
    // Several small groups in a wave: with few edges a lane per replica and objective reads
    // out, since the whole wave would take those one after the other (calls of 60 steps: 2
    // nodes, m = 8, 3200 replicas 122 -> 19 us; 12 nodes, m = 3, 10 000 27 -> 22; at the line,
    // complete 12 nodes, m = 3, 3200 no difference).
    const bool flat = shape == 0 && a.per_block > 1 &&
                      p.E <= 4 * std::min<int64_t>(a.per_block, a.groups) * V * p.m;
    const dim3 grid((unsigned)blocks);
    const dim3 block(NT);
    if (full) {
        launch_group_full(shape, dsb, p.max_degree, flat, grid, block, a, st);
    } else if (V == 1) {
        launch_group_v1(shape, dsb, p.max_degree, flat, grid, block, a, st);
    } else {
#define QAIA_V4(SHAPE, NTMAX, NPT, LONG)                                                                     \
    case SHAPE:                                                                                              \
        if (dsb) launch_group_deg<NTMAX, NPT, 4, true, false, LONG>(p.max_degree, flat, grid, block, a, st); \
        else launch_group_deg<NTMAX, NPT, 4, false, false, LONG>(p.max_degree, flat, grid, block, a, st);    \
        break;
        switch (shape) {
            QAIA_V4(0, 64, 1, true)
            QAIA_V4(1, 64, 2, true)
            QAIA_V4(2, 64, 4, false)
            QAIA_V4(3, 256, 2, false)
            QAIA_V4(4, 256, 4, false)
            QAIA_V4(5, 512, 1, true)
            default:
            QAIA_V4(6, 512, 2, true)
        }
#undef QAIA_V4
    }
    QAIA_HIP(hipGetLastError());
}

}  // namespace qaia
