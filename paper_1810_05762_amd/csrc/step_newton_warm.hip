// Step kernel family: Newton / Krylov solver, warm-started.
#include "step_variants_impl.hpp"

template const void* sim355::step_variant_of<0, 1, 1>(int, int, bool);
