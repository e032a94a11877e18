// The GMRES launchers of basis-size bounds above 8 for storage half_t, compute double.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(, half_t, double)
}  // namespace mprk
