// The GMRES launchers of basis-size bounds above 8 for storage double, compute double.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(, double, double)
}  // namespace mprk
