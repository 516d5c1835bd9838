// The compiled forms of the step kernel.  One translation unit per family (plain, capsule-capsule
// collisions, warm start, both, Newton, Newton with warm start), so that they compile side by side;
// sim.hip asks for the entry point that suits a launch and starts it by address.
#pragma once

namespace sim355 {

// Envs per workgroup that have a form of their own (index arithmetic and LDS offsets fixed at
// compile time); any other number runs the general form, which takes it from the launch arguments
// and is a quarter to a third slower (300 self-colliding humanoids with the warm start: 149 us as
// workgroups of 3, 119 us of 4, 111 us of 2).  The Newton families end at 8 (a contact thread per slot).
// One env per workgroup is the library's own choice only with collisions (room in the contact queue)
// and where two do not fit; elsewhere a caller asks for it.  All forms of a family give the same bits
// (robots that the whole workgroup solves with Newton's method aside), so size and speed alone decide.
constexpr bool step_compiled_envs(int E, bool newton) {
  return (E == 16 && !newton) || E == 8 || E == 4 || E == 2 || E == 1;
}

// Entry point for E envs and `threads` threads per workgroup; `few`: no body belongs to more than
// four joints.  Instantiated once per family.
template <int PC, int WS, int NS>
const void* step_variant_of(int E, int threads, bool few);

}  // namespace sim355
