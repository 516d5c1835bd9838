// Definition of step_variant_of: included by the one source file of each family.
#pragma once
#include "step_kernel.hpp"
#include "step_variants.hpp"

namespace sim355 {

template <int PC, int WS, int NS>
const void* step_variant_of(int E, int threads, bool few) {
  auto entry = [](auto kern) { return reinterpret_cast<const void*>(kern); };
  if (!few) return entry(&step_kernel<0, kMaxBodyJoints, PC, kThreads, WS, NS>);
  if constexpr (PC == 0 && WS == 0 && NS == 0) {
    if (threads == kThreadsWide) return entry(&step_kernel<16, 4, 0, kThreadsWide>);
  } else if constexpr (NS == 0) {
    if (E == 16) return entry(&step_kernel<16, 4, PC, kThreads, WS, NS, joint_lanes(16, true, PC != 0, false)>);
  }
  if (E == 8) return entry(&step_kernel<8, 4, PC, kThreads, WS, NS, joint_lanes(8, true, PC != 0, NS != 0)>);
  if (E == 4) return entry(&step_kernel<4, 4, PC, kThreads, WS, NS, joint_lanes(4, true, PC != 0, NS != 0)>);
  if (E == 2) return entry(&step_kernel<2, 4, PC, kThreads, WS, NS, joint_lanes(2, true, PC != 0, NS != 0)>);
  if (E == 1) return entry(&step_kernel<1, 4, PC, kThreads, WS, NS, joint_lanes(1, true, PC != 0, NS != 0)>);
  return entry(&step_kernel<0, 4, PC, kThreads, WS, NS>);
}

}  // namespace sim355
