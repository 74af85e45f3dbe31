// The persistent GEMM kernel for E4M3 operands.
#include "gemm_persistent.h"

namespace hero_gemm {
HERO_PERSISTENT_8BIT(HERO_F8E4M3, HERO_F8E4M3)
}  // namespace hero_gemm
