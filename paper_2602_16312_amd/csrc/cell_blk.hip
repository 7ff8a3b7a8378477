// Cell kernels on stored blocks, of nodal levels and whole.
#include "cell_launch.hpp"

namespace dgmg {

DGMG_CELL_LAUNCHERS(float, GEO_BLK)
DGMG_CELL_LAUNCHERS(float, GEO_BLD)
DGMG_CELL_LAUNCHERS(double, GEO_BLD)
DGMG_CELL_LAUNCHERS(double, GEO_BLK)

}  // namespace dgmg
