// Step kernel family: capsule-capsule collisions and warm-started rows.
#include "step_variants_impl.hpp"

template const void* sim355::step_variant_of<1, 1, 0>(int, int, bool);
