// Step kernel family: terrain contacts, Jacobi sweeps.
#include "step_variants_impl.hpp"

template const void* sim355::step_variant_of<0, 0, 0>(int, int, bool);
