// The ring kernel with E4M3 operands (the FP8 variant, paper Sec. 2.1).
#include "gemm_ring.h"

namespace hero_gemm {
template hero_status launch_ring_part<HERO_F8E4M3>(GemmArgs, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_REQUANT, HERO_F8E4M3, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_GELU_REQUANT, HERO_F8E4M3, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_BF16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_F16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_F16, HERO_F16>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1>(const GemmArgs&, RingForm, hipStream_t);
template hero_status launch_ring<HERO_F8E4M3, HERO_EPI_DEQUANT_GELU, HERO_F16, -1>(const GemmArgs&, RingForm, hipStream_t);
}  // namespace hero_gemm
