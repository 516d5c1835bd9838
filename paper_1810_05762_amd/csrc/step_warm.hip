// Step kernel family: warm-started rows.
#include "step_variants_impl.hpp"

template const void* sim355::step_variant_of<0, 1, 0>(int, int, bool);
