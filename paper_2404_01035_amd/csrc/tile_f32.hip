// Plain 2D tile kernels (several steps per launch), F32.
#include "tile2d.hpp"

namespace mp {
template int call_tile<float, false>(const StepLaunch&, const Coef<float>&, const CoefX<float>*, KernelCall&);
}
