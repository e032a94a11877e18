// The GMRES launchers of basis-size bounds above 8 for storage float, compute double.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(, float, double)
}  // namespace mprk
