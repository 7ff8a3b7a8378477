// Cell kernels on bilinear and trilinear cells.
#include "cell_launch.hpp"

namespace dgmg {

DGMG_CELL_LAUNCHERS(float, GEO_MAP)
DGMG_CELL_LAUNCHERS(double, GEO_MAP)
DGMG_CELL_RHS(GEO_MAP)

}  // namespace dgmg
