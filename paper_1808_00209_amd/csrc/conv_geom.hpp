// Geometry of one conv launch (stride 1), without any HIP header: the plans
// of the launchers (tile_plans.hpp) are host code that needs nothing else.
#pragma once

#include <stdint.h>

namespace bnn {

// Cw, Fw: words of C and F bits; Ho, Wo: outputs before pooling; Hp, Wp:
// stored bits.
struct ConvGeom {
  int32_t N, H, W, C, F, KH, KW, pad, pool;
  int32_t Cw, Fw, Ho, Wo, Hp, Wp;
};

}  // namespace bnn
