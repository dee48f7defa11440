// Moment-form adjoint edge stage (device/adjoint.hip): which plans it covers, its slot groups and source.
#pragma once

#include <string>
#include <vector>

#include "plan.h"

namespace sobek {

// channels [U0, U0 + 16 UT) of input irrep a, UT its group's; its 2 l + 1 slots start at `slot`
struct AdjJob {
  int a, U0, slot;
};
// slots formed together, one 16-channel tile at a time (jobs of one width, UT tiles)
struct AdjGroup {
  int UT = 0, slots = 0;
  std::vector<AdjJob> jobs;
};

// fully connected plans with K = 16, lmax of 2 or more, input multiplicities in multiples of 16 and at least 30
// steps (channel tile, pair of m_y)
bool adjoint_plan(const Plan& p);
std::vector<AdjGroup> adjoint_groups(const Plan& p);
// text that follows generate_split_source's and emit_sh's
std::string generate_adjoint_source(const Plan& p);

}  // namespace sobek
