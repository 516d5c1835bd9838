// Step kernel family: capsule-capsule collisions.
#include "step_variants_impl.hpp"

template const void* sim355::step_variant_of<1, 0, 0>(int, int, bool);
