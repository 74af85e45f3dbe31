// The persistent GEMM kernel for INT8 operands.
#include "gemm_persistent.h"

namespace hero_gemm {
HERO_PERSISTENT_8BIT(HERO_I8, HERO_I8)
template hero_status launch_persistent_tile<HERO_I8, HERO_EPI_RAW_I32, HERO_I32, -1>(const GemmArgs&, int, hipStream_t);
template hero_status launch_persistent_part<HERO_I8>(const GemmArgs&, int, hipStream_t);
}  // namespace hero_gemm
