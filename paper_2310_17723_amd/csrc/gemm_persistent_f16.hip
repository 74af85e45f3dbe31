// The persistent GEMM kernel for float16 operands.
#include "gemm_persistent.h"

namespace hero_gemm {
HERO_PERSISTENT_16BIT(HERO_F16)
}  // namespace hero_gemm
