// What the kernels of the layer product H = Z W (Section 3, Eq. 1) on the fp64 matrix cores share.
#pragma once
#include "common.hpp"

namespace csgs {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32;   // k per chunk

}  // namespace csgs
