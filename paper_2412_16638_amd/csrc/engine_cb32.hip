// Instantiation of the LP-solve engine for storage float, compute double (GMRES bounds above 8:
// engine_cb32_arnoldi.hip).
// FP64 arithmetic over FP32 storage is a compressed-basis Krylov variant: the basis and every Krylov
// vector stored in the low precision, all arithmetic, dot products and updates in FP64.
#include "engine.hpp"

namespace mprk {
MPRK_ARNOLDI_LARGE(extern, float, double)
Engine* make_engine_cb32() { return new EngineT<float, double>(); }
}  // namespace mprk
