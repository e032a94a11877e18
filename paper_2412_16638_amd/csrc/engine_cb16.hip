// Instantiation of the LP-solve engine for storage half_t, compute double (GMRES bounds above 8:
// engine_cb16_arnoldi.hip).
// FP64 arithmetic over FP16 storage is a compressed-basis Krylov variant: the basis and every Krylov
// vector stored in the low precision, all arithmetic, dot products and updates in FP64.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(extern, half_t, double)
Engine* make_engine_cb16() { return new EngineT<half_t, double>(); }
}  // namespace mprk
