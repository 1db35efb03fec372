// Noise-injecting and tracing instantiations of the one-spin-per-lane sparse kernel.
#include "group.hpp"

namespace qaia {

void launch_group_full(int shape, bool dsb, int maxdeg, bool flat, dim3 grid, dim3 block, const GroupArgs &a, hipStream_t st) {
#define QAIA_GROUP(SHAPE, NTMAX, NPT)                                                                 \
    case SHAPE:                                                                                       \
        if (dsb) launch_group_deg<NTMAX, NPT, 1, true, true, true>(maxdeg, flat, grid, block, a, st); \
        else launch_group_deg<NTMAX, NPT, 1, false, true, true>(maxdeg, flat, grid, block, a, st);    \
        break;
    switch (shape) {
        QAIA_GROUP(0, 64, 1)
        QAIA_GROUP(1, 64, 2)
        QAIA_GROUP(3, 256, 2)
        default:
        QAIA_GROUP(4, 256, 4)
    }
#undef QAIA_GROUP
}

}  // namespace qaia
