// The persistent GEMM kernel for bfloat16 operands.
#include "gemm_persistent.h"

namespace hero_gemm {
HERO_PERSISTENT_16BIT(HERO_BF16)
}  // namespace hero_gemm
