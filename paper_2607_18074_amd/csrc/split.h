// Channel products on split operands (device/split.hip): which plans they cover and the generated source.
#pragma once

#include <algorithm>
#include <string>

#include "plan.h"

namespace sobek {

// fp32 fully connected plans with multiplicities in multiples of 4: channel products on split operands
bool split_plan(const Plan& p);
int split_bn(int C);   // column tile of a group's products
// Splits of a group's weight-gradient rows at most: about 512 blocks of 128 x 64 tiles.
inline int ga_max_splits(const Plan& p, const Group& g) {
  const int bn = g.C <= 16 ? 16 : g.C <= 32 ? 32 : 64;
  const int64_t tiles = ((g.D + (p.vec4 ? 127 : 63)) / (p.vec4 ? 128 : 64)) * ((g.C + bn - 1) / bn);
  return (int)std::max<int64_t>(1, std::min<int64_t>((512 + tiles - 1) / tiles, 64));
}
// Device code for split operands and, for plans split_plan covers, the products' entry points.
std::string generate_split_source(const Plan& p);

}  // namespace sobek
