// The ring kernel with 16-bit operands (the 16-bit side of a switched module, paper Sec. 2.3, Table 1): K that ends in half a slab.
#include "gemm_ring.h"

namespace hero_gemm {
HERO_RING_16BIT(HERO_BF16, true)
HERO_RING_16BIT(HERO_F16, true)
}  // namespace hero_gemm
