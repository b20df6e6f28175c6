// Plain 2D tile kernels (several steps per launch), F64.
#include "tile2d.hpp"

namespace mp {
template int call_tile<double, false>(const StepLaunch&, const Coef<double>&, const CoefX<double>*, KernelCall&);
}
