"""Which kernel a product runs, asked of the library's own rule (include/hero_debug.h); nothing is launched."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

FORMS = ["32x32/8", "32x32/4", "32x64/2", "32x64/4", "64x32/4", "64x64/2", "64x64", "128x64/2", "128x64", "128x128"]
DTYPES = [torch.int8, torch.float8_e4m3fn, torch.bfloat16, torch.float16]


def kernel(dt, M, N, kb, **kw):
    k = pkg.load().hero_gemm_kernel(dt, M, N, kb // dt.itemsize, **kw)
    return FORMS[k - 16] if k >= 16 else k


@pytest.mark.parametrize("dt", DTYPES)
def test_half_slab_keeps_the_ring(dt):
    """A K of an odd number of 64-byte pieces runs what the next whole slab would: the direct-to-LDS ring, not the kernel that
    stages through registers (measured 1.7 to 3.5 times as long for few rows)."""
    for N, K in ((768, 768), (1024, 1024), (4096, 2048), (4096, 4096), (12288, 4096), (4096, 16384)):
        for M in (1, 16, 64, 100, 256, 512, 1000):
            whole = kernel(dt, M, N, K + 128)
            if isinstance(whole, str):
                assert kernel(dt, M, N, K + 64) == whole, (M, N, K)
    assert kernel(dt, 2048, 4096, 4160) == "128x128"            # no form for a whole slab either: 128 x 128 tiles
    assert kernel(dt, 2048, 4096, 2112) == 0                    # .. through registers while K is short
    assert kernel(dt, 4096, 4096, 2112) == (1 if dt == torch.int8 else 0)
    # rows too far apart for 32-bit offsets: registers, the small tile for few rows
    assert kernel(dt, 64, 4096, 4096, lda=1 << 24) == 3 and kernel(dt, 4096, 4096, 1024, lda=1 << 24) in (0, 1)


def test_split_scratch_is_asked_for_where_k_splits():
    """hero_int8_gemm_workspace_bytes: 0 for a shape that runs in one pass (so that the entry point with the built-in scratch
    takes it, whatever its size), a size for one that splits, K of whole slabs or not."""
    need = pkg.load().hero_int8_gemm_workspace_bytes
    for M, N, K in ((128, 16384, 8192), (65, 8256, 16384), (100, 12288, 8192), (64, 16384, 8192), (129, 4096, 16384), (64, 4096, 4096)):
        assert need(M, N, K) == 0, (M, N, K)
    for M, N, K in ((1, 512, 8192), (64, 4096, 16384), (64, 8192, 8192), (128, 8192, 8192), (100, 2304, 8192), (33, 4096, 8256)):
        assert need(M, N, K) >= 2 * M * N * 4, (M, N, K)


@pytest.mark.parametrize("dt", [torch.int8, torch.float8_e4m3fn])
def test_narrow_tiles_are_not_for_two_rounds_of_8_bit_results(dt):
    """128 x 64 tiles write half a line of an 8-bit result: beyond the first round of tiles the persistent kernel takes it (measured
    8-30 % ahead), likewise with a GELU epilogue; 16-bit results with a short K stay."""
    PERSISTENT = (7, 8)
    for M, N, K in ((8192, 1024, 1024), (5400, 768, 768), (10240, 768, 768), (2048, 3072, 1024), (2500, 2304, 768), (1500, 3072, 1024)):
        assert kernel(dt, M, N, K, epi=HB.EPI_REQUANT) in PERSISTENT, (M, N, K)
        assert kernel(dt, M, N, K) == "128x64", (M, N, K)
    for M, N, K in ((2048, 4096, 1024), (2500, 3072, 768), (1800, 4096, 1024)):
        assert kernel(dt, M, N, K, epi=HB.EPI_GELU_REQUANT) in PERSISTENT, (M, N, K)
    assert kernel(dt, 4096, 1024, 1024, epi=HB.EPI_REQUANT) == "128x128"
    assert kernel(dt, 3000, 1024, 1024, epi=HB.EPI_REQUANT) == "128x64"


def test_e4m3_of_a_long_k_and_several_rounds_takes_small_tiles():
    """Three rounds of 128 x 128 tiles for one of 256 x 256: ahead for E4M3 from the second large round on (up to 12 %), not for INT8."""
    f8, i8 = torch.float8_e4m3fn, torch.int8
    for M, N, K in ((3072, 12288, 4096), (6144, 4096, 4096), (1500, 16384, 4096), (12000, 2048, 8192)):
        assert kernel(f8, M, N, K) == 8 and kernel(i8, M, N, K) == 7, (M, N, K)
    for M, N, K in ((768, 12288, 4096), (2500, 16384, 4096), (16384, 12288, 4096)):
        assert kernel(f8, M, N, K) == 7, (M, N, K)


@pytest.mark.parametrize("dt", DTYPES)
def test_small_tiles_of_a_long_k_while_all_are_resident(dt):
    """257 to 448 tiles of 128 x 128 (two on some CUs) behind a K of 8 KB or more: ahead of tiles of 160 rows (weights from memory, up to 15 % for 16 bits), which
    would leave most CUs without work.  The taller ones beyond that, and with four or eight full rows of tiles (up to 14 % ahead)."""
    for M, N, kb in ((5943, 768, 16384), (301, 12288, 8192), (4637, 1024, 8192), (431, 12288, 8192), (1700, 4096, 16384), (1313, 4096, 16384), (1310, 4096, 32768)):
        assert kernel(dt, M, N, kb) == 8, (M, N, kb)
    for M, N, kb in ((705, 12288, 8192), (633, 16384, 8192), (2438, 4096, 32768), (505, 12288, 8192), (525, 12288, 8192), (1000, 8192, 8192), (2040, 4096, 32768)):
        if dt != torch.float8_e4m3fn:                               # (which has no tiles of 160 rows)
            assert kernel(dt, M, N, kb) == 7, (M, N, kb)


@pytest.mark.parametrize("dt", DTYPES)
def test_few_rows_of_many_columns_keep_small_tiles(dt):
    """A product of at most 64 rows never runs tiles of 128 or 256 rows, however many columns it has."""
    for N in (33000, 36864, 50304, 131072):
        for kb in (1024, 4096, 8192):
            assert kernel(dt, 1, N, kb) == {1024: "64x64", 4096: "32x64/2", 8192: "32x64/4"}[kb]
            assert kernel(dt, 33, N, kb) == kernel(dt, 64, N, kb) == "64x64"


def test_ring_test_shapes_reach_every_form():
    """The shapes of the ring kernel's GPU tests select every form, with whole slabs and with half a one, for every type."""
    from test_gpu_gemm_ring import SHAPES
    for dt in DTYPES:
        for half in (0, 64):
            assert set(FORMS) <= {kernel(dt, M, N, kb) for M, N, kb in SHAPES if kb % 128 == half}
