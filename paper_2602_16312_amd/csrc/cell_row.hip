// Cell kernels on whole blocks of 64 rows.
#include "cell_launch.hpp"

namespace dgmg {

DGMG_CELL_LAUNCHERS(float, GEO_ROW)
DGMG_CELL_LAUNCHERS(double, GEO_ROW)

}  // namespace dgmg
