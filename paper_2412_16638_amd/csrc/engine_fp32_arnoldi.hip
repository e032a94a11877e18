// The GMRES launchers of basis-size bounds above 8 for storage float, compute float.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(, float, float)
}  // namespace mprk
