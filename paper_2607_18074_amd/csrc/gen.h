// Pieces of the kernel generator shared by its translation units.
#pragma once

#include <sstream>
#include <string>
#include <utility>
#include <vector>

#include "plan.h"

namespace sobek {

struct PairTerm { int my; double c; };

// Sparse structure of a path's coupling: the (m_i, m_o) pairs with a nonzero
// coefficient, each with its (m_y, c) terms.
struct PathTerms {
  std::vector<std::pair<int, int>> pairs;
  std::vector<std::vector<PairTerm>> terms;
};
PathTerms path_terms(const Path& q);

std::string fl(double v);                       // float literal
void emit_sh(std::ostringstream& o, int lmax);  // spherical harmonics and their derivatives

}  // namespace sobek
