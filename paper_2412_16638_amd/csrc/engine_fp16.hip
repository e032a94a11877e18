// Instantiation of the LP-solve engine for storage half_t, compute float (GMRES bounds above 8:
// engine_fp16_arnoldi.hip).
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(extern, half_t, float)
Engine* make_engine_fp16() { return new EngineT<half_t, float>(); }
}  // namespace mprk
