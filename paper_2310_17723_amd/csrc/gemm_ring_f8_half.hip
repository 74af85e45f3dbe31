// The ring kernel with E4M3 operands (the FP8 variant, paper Sec. 2.1): K that ends in half a slab.
#include "gemm_ring.h"

namespace hero_gemm {
HERO_RING_8BIT(HERO_F8E4M3, HERO_F8E4M3, true)
}  // namespace hero_gemm
