/* hero_debug.h -- test and tuning hooks of libhero.  NOT part of the product interface (include/hero.h): the
 * product entry points choose their kernel from the problem size alone and read no environment variable.
 * Each hook is the entry point of the same name without the suffix, with one more argument that forces the
 * kernel; arguments, constraints, error behaviour and results are otherwise identical (for INT8 operands every
 * kernel gives bit-identical results; for FP8 and BF16 operands the order of the fp32 accumulation, and with it
 * the last bits, depends on the tile).  A forced kernel that cannot run the shape falls back to its closest
 * relative; an unknown tile code returns HERO_ERR_UNSUPPORTED.  All pointers are device pointers. */
#ifndef HERO_DEBUG_H
#define HERO_DEBUG_H

#include "hero.h"

#ifdef __cplusplus
extern "C" {
#endif

/* GeMM^quant (Sec. 2.1, 2.2.2, 2.2.3) with the kernel forced.  tile: 0 = 128x128 tile staged through registers,
 * 1 = 256x256 direct-to-LDS, one tile per workgroup, 2 = the ring kernel (small and middling problems), 7 = 256x256
 * persistent, 8 = 128x128 persistent (two workgroups per CU), 10 / 11 / 12 = persistent of 224 / 192 / 160 rows by 256 columns;
 * 9, the code of a former kernel, runs as 7.  The persistent kernels, here and below, run every M and N whose K is a multiple of 128 bytes,
 * 256 or more (160 rows: 384 or more, else as 192), and whose rows lie less than 16 MB apart.  Never splits K. */
hero_status hero_int8_gemm_tile(const int8_t* A, int64_t lda, const float* a_row_scale,
                                const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                hero_epilogue epi, const float* out_col_scale,
                                void* C, hero_dtype c_dt, int64_t ldc,
                                int64_t M, int64_t N, int64_t K, void* stream, int tile);

/* The FP8 variant (Sec. 2.1).  tile: 0 = 128x128 staged through registers, 7 / 8 / 11 = persistent 256x256 / 128x128 / 192x256. */
hero_status hero_fp8_gemm_tile(const void* A, int64_t lda, const float* a_row_scale,
                               const void* Bt, int64_t ldb, const float* b_col_scale,
                               const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                               hero_epilogue epi, const float* out_col_scale,
                               void* C, hero_dtype c_dt, int64_t ldc,
                               int64_t M, int64_t N, int64_t K, void* stream, int tile);

/* The 16-bit side of a switched module (Sec. 2.3, Table 1; hero_hp_gemm).  tile: 0 = the kernels for smaller problems,
 * 7 / 8 / 10 / 11 / 12 = the persistent 256x256 / 128x128 / 224x256 / 192x256 / 160x256 kernel. */
hero_status hero_hp_gemm_tile(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                              const float* bias, const void* residual, int64_t ldr, int gelu,
                              void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, hero_dtype dt, void* stream, int tile);

/* Which kernel hero_int8_gemm (dt HERO_I8), hero_fp8_gemm (HERO_F8E4M3) or hero_hp_gemm (HERO_BF16 / HERO_F16) runs for a
 * product without residual and without scratch, with the epilogue `epi`.  Returns a tile code as above (7 for every height of the persistent kernel's 256 columns; 3 = 64x64 tile
 * staged through registers, 4 = the weight-streaming kernel of few rows) or, for the ring kernel, 16 + its form: 0 = 32x32 with eight K groups, 1 = 32x32 with four,
 * 2 / 3 = 32x64 with two / four, 4 = 64x32 with four, 5 = 64x64 with two, 6 = 64x64, 7 = 128x64 with two, 8 = 128x64,
 * 9 = 128x128.  Launches nothing. */
int hero_gemm_kernel(hero_dtype dt, hero_epilogue epi, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb);

#ifdef __cplusplus
}
#endif
#endif /* HERO_DEBUG_H */
