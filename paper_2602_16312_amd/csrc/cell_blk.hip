// Cell kernels on stored blocks of nodal levels.
#include "cell_launch.hpp"

namespace dgmg {

DGMG_CELL_LAUNCHERS(float, GEO_BLK)
DGMG_CELL_LAUNCHERS(double, GEO_BLK)

}  // namespace dgmg
