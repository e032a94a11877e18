// The GMRES launchers of basis-size bounds above 8 for storage half_t, compute float.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(, half_t, float)
}  // namespace mprk
