// bz_plan.hpp -- what the host decides before a launch, from shapes and options
// alone (no device calls, so that it is checked on the CPU).
#pragma once
#include <stdint.h>

#include "bz_units.hpp"

namespace bz {

// Workgroups per compute unit of the kernel without tables, at most.  Its
// registers allow one more over F_7, but a wider grid lets more stages start
// at once, whose work is thrown away when an earlier one ends the run (F_7
// without tables, [48, 12] 66.8 us with three, 89.0 with four; [66, 11] 81.4
// and 92.0; [108, 9], four words, 131.1 with two, 136.6 with three).
inline int prefix_groups(int p, int W) { return p == 3 ? (W <= 2 ? 5 : 4) : W == 1 ? 4 : W == 2 ? 3 : 2; }

}  // namespace bz
