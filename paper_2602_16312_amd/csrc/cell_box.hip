// Cell kernels on identical boxes.
#include "cell_launch.hpp"

namespace dgmg {

unsigned cell_groups(int geo, int b, int n) {
    const int nc = cells_per_group(geo, b, n, false);
    return (unsigned)((n + nc - 1) / nc);
}

DGMG_CELL_LAUNCHERS(float, GEO_BOX)
DGMG_CELL_LAUNCHERS(double, GEO_BOX)
DGMG_CELL_RHS(GEO_BOX)

}  // namespace dgmg
