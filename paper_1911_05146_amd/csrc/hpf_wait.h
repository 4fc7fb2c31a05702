// The bound on the waits of the register-resident kernels for their partners' words.  Plain C++ (constexpr functions are compiled for both
// sides), so that it can be tested on the host.
#pragma once

namespace hpf {

constexpr unsigned RES_SPIN_LIMIT = 1u << 19;

// Looks in vain that one collection has left, over all its chunks of members together: with a limit per chunk a work-group
// without partners would hold its CU for as many limits as there are chunks (four for 64 images in the backward of 128-64 blocks).
struct SpinBudget {
  unsigned spins = 0;
  constexpr bool spent() const { return spins > RES_SPIN_LIMIT; }
  constexpr bool again() { return ++spins <= RES_SPIN_LIMIT; }   // after a look in vain: may another one follow?
};
// The chunks of a collection: for (int b = 0; more_chunks(b, nmem, budget); b += chunk)
constexpr bool more_chunks(int b, int nmem, const SpinBudget& budget) { return b < nmem && !budget.spent(); }

}  // namespace hpf
