// Instantiation of the LP-solve engine for storage float, compute float (GMRES bounds above 8:
// engine_fp32_arnoldi.hip).
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(extern, float, float)
Engine* make_engine_fp32() { return new EngineT<float, float>(); }
}  // namespace mprk
