// One-replica instantiations of the one-spin-per-lane sparse kernel.
#include "group.hpp"

namespace qaia {

void launch_group_v1(int shape, bool dsb, int maxdeg, bool flat, dim3 grid, dim3 block, const GroupArgs &a, hipStream_t st) {
#define QAIA_GROUP(SHAPE, NTMAX, NPT, LONG)                                                            \
    case SHAPE:                                                                                        \
        if (dsb) launch_group_deg<NTMAX, NPT, 1, true, false, LONG>(maxdeg, flat, grid, block, a, st); \
        else launch_group_deg<NTMAX, NPT, 1, false, false, LONG>(maxdeg, flat, grid, block, a, st);    \
        break;
    switch (shape) {
        QAIA_GROUP(0, 64, 1, true)
        QAIA_GROUP(1, 64, 2, true)
        QAIA_GROUP(2, 64, 4, false)
        QAIA_GROUP(3, 256, 2, false)
        QAIA_GROUP(4, 256, 4, false)
        QAIA_GROUP(5, 512, 1, true)
        default:
        QAIA_GROUP(6, 512, 2, true)
    }
#undef QAIA_GROUP
}

}  // namespace qaia
