// The ring kernel with 16-bit operands (the 16-bit side of a switched module, paper Sec. 2.3, Table 1).
#include "gemm_ring.h"

namespace hero_gemm {
#define HERO_RING_HP(DT) \
    template hero_status launch_ring_part<DT>(GemmArgs, RingForm, hipStream_t); \
    template hero_status launch_ring<DT, HERO_EPI_DEQUANT, DT, -1>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring<DT, HERO_EPI_DEQUANT, DT, DT>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring<DT, HERO_EPI_DEQUANT_GELU, DT, -1>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring<DT, HERO_EPI_DEQUANT_GELU, DT, DT>(const GemmArgs&, RingForm, hipStream_t);
HERO_RING_HP(HERO_BF16)
HERO_RING_HP(HERO_F16)
#undef HERO_RING_HP
}  // namespace hero_gemm
