// The compiled forms of the step kernel.  One translation unit per family (plain, capsule-capsule
// collisions, warm start, both, Newton, Newton with warm start), so that they compile side by side;
// sim.hip asks for the entry point that suits a launch and starts it by address.
#pragma once

namespace sim355 {

// Envs per workgroup that have a form of their own (index arithmetic and LDS offsets fixed at
// compile time); any other number runs the general form, which takes it from the launch arguments
// and is a quarter to a third slower (300 self-colliding humanoids with the warm start: 137 us as
// workgroups of 3, 104 us of 4, 100 us of 2).  The Newton families end at 8 (a contact thread per slot).
// One env per workgroup is the library's own choice only with collisions (room in the contact queue)
// and where two do not fit; elsewhere a caller asks for it.  All forms of a family give the same bits
// (robots that the whole workgroup solves with Newton's method aside), so size and speed alone decide.
constexpr bool step_compiled_envs(int E, bool newton) {
  return (E == 16 && !newton) || E == 8 || E == 4 || E == 2 || E == 1;
}

// Lanes that relax one joint in the form for E envs per workgroup.  More lanes make a wavefront's chain shorter and
// give the SIMDs more wavefronts that hold each other up.  Cycles per sweep: up to 4 envs four lanes (64 humanoids
// 747, with two 789; 1024 765 and 834), which fill no more wavefronts than there are SIMDs (three with humanoids);
// 8 envs two lanes (1500 humanoids 1003, with one 1186; that collide in groups of 8 1267 and 1440); collisions of 16
// envs in 512 threads one (groups of 4: 1765, with two 2015); of up to 4 envs two, as four win nothing beside the
// pairs' own lanes (groups of 4: 1077 and 1093).
constexpr int joint_lanes(int E, bool few, bool pairs, bool newton) {
  if (!few || newton) return 2;
  if (pairs) return E == 16 ? 1 : 2;
  return E == 4 || E == 2 || E == 1 ? 4 : 2;
}

// Entry point for E envs and `threads` threads per workgroup; `few`: no body belongs to more than
// four joints.  Instantiated once per family.
template <int PC, int WS, int NS>
const void* step_variant_of(int E, int threads, bool few);

}  // namespace sim355
