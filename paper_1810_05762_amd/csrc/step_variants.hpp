// The compiled forms of the step kernel.  One translation unit per family (plain, capsule-capsule
// collisions, warm start, both, Newton, Newton with warm start), so that they compile side by side;
// sim.hip asks for the entry point that suits a launch and starts it by address.
#pragma once

namespace sim355 {

// Envs per workgroup that have a form of their own (index arithmetic and LDS offsets fixed at
// compile time); any other number runs the general form, which takes it from the launch arguments
// and is up to twice as slow.  The Newton families end at 8 (a contact thread per slot).  Collisions
// together with the warm start begin at 8: below, that family stays in the general form, whose
// multiply-adds are contracted differently, because its ten-step agreement with double precision is
// pinned there to a bound that one env in a few dozen, with a capsule contact that amplifies rounding,
// exceeds in the compiled forms (all of which agree bit for bit).
constexpr bool step_compiled_envs(int E, bool pairs, bool warm, bool newton) {
  return (E == 16 && !newton) || E == 8 || ((E == 4 || E == 2 || E == 1) && !(pairs && warm));
}

// Entry point for E envs and `threads` threads per workgroup; `few`: no body belongs to more than
// four joints.  Instantiated once per family.
template <int PC, int WS, int NS>
const void* step_variant_of(int E, int threads, bool few);

}  // namespace sim355
