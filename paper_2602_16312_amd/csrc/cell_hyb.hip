// Cell kernels on Q1 cells with stored cell blocks and faces' metric data.
#include "cell_launch.hpp"

namespace dgmg {

DGMG_CELL_LAUNCHERS(float, GEO_HYB)
DGMG_CELL_LAUNCHERS(double, GEO_HYB)

}  // namespace dgmg
