// General 2D tile kernels (several steps per launch), F32.
#include "tile2d.hpp"

namespace mp {
template int call_tile<float, true>(const StepLaunch&, const Coef<float>&, const CoefX<float>*, KernelCall&);
}
