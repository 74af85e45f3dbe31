// The ring kernel with 16-bit operands (the 16-bit side of a switched module, paper Sec. 2.3, Table 1).
#include "gemm_ring.h"

namespace hero_gemm {
HERO_RING_16BIT(HERO_BF16, false)
HERO_RING_16BIT(HERO_F16, false)
}  // namespace hero_gemm
