// The ring kernel with INT8 operands (paper Sec. 2.1, 2.2.2, 2.2.3).
#include "gemm_ring.h"

namespace hero_gemm {
template hero_status launch_ring_part<HERO_I8>(GemmArgs, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_RAW_I32, HERO_I32, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_REQUANT, HERO_I8, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_GELU_REQUANT, HERO_I8, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT, HERO_BF16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT, HERO_F16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT, HERO_F16, HERO_F16>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_I8, HERO_EPI_DEQUANT_GELU, HERO_F16, -1>(const GemmArgs&, RingForm, hipStream_t);
}  // namespace hero_gemm
