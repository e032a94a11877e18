// Instantiation of the LP-solve engine for storage double, compute double (GMRES bounds above 8:
// engine_fp64_arnoldi.hip).
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(extern, double, double)
Engine* make_engine_fp64() { return new EngineT<double, double>(); }
}  // namespace mprk
