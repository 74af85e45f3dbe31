// The ring kernel with INT8 operands (paper Sec. 2.1, 2.2.2, 2.2.3).
#include "gemm_ring.h"

namespace hero_gemm {
HERO_RING_8BIT(HERO_I8, HERO_I8, false)
template hero_status launch_ring_slabs<HERO_I8, HERO_EPI_RAW_I32, HERO_I32, -1, false>(const GemmArgs&, RingForm, hipStream_t);
}  // namespace hero_gemm
