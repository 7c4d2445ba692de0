"""Which kernel a GEMM goes to, by its sizes and strides (no GPU)."""

import pytest

from paper_2308_15762_amd import hanayo as hn

WAVE_64x64, WAVE_32x32, WAVE_96x64, WAVE_32x64, ALU = 0, 1, 12, 13, 14


def choice(M, N, K, lda=None, ldc=None, b_t=True, epilogue=hn.EPI_NONE, dtype=hn.BF16, a_t=False):
    return hn.hanayo_op_gemm_kernel(dtype, M, N, K, lda or (M if a_t else K), N if b_t else K, ldc or N, a_t, b_t, epilogue)


def test_choice_reports_forced_kernels_and_refuses_what_the_call_refuses():
    for config in (0, 1, 7, 9, 10, 11):
        hn.hanayo_op_gemm_config(config)
        try:
            assert choice(1024, 1024, 1024) == config
        finally:
            hn.hanayo_op_gemm_config(-1)
    assert choice(100, 100, 100) == ALU   # rows of 200 bytes
    for bad in (dict(M=0), dict(epilogue=99), dict(lda=8), dict(dtype=7)):
        with pytest.raises(hn.HanayoError):
            choice(**{**dict(M=64, N=64, K=64), **bad})


@pytest.mark.parametrize("b_t", [True, False])
def test_lane_offsets_stay_within_31_bits(b_t):
    """A 96-row tile spans 96 rows of A with 32-bit offsets, the square ones 64."""
    M, N, K = 200, 5000, 1024
    assert choice(M, N, K, b_t=b_t) == WAVE_96x64
    last = (2 ** 31 - 1) // (96 * 2) // 8 * 8
    assert choice(M, N, K, lda=last, b_t=b_t) == WAVE_96x64
    assert choice(M, N, K, lda=last + 8, b_t=b_t) in (WAVE_64x64, WAVE_32x32, WAVE_32x64)
    last = (2 ** 31 - 1) // (64 * 2) // 8 * 8
    assert choice(M, N, K, lda=last, b_t=b_t) in (WAVE_64x64, WAVE_32x32, WAVE_32x64)
    assert choice(M, N, K, lda=last + 8, b_t=b_t) not in (WAVE_64x64, WAVE_32x32, WAVE_32x64, WAVE_96x64)


@pytest.mark.parametrize("b_t", [True, False])
@pytest.mark.parametrize("M, N, K, kernel", [
    (1536, 768, 1024, WAVE_96x64), (1527, 768, 3072, WAVE_96x64), (1441, 760, 2056, WAVE_96x64), (700, 1536, 1608, WAVE_96x64),
    (777, 640, 2560, WAVE_32x64), (769, 632, 520, WAVE_32x64), (1024, 512, 2048, WAVE_32x64), (96, 3840, 1288, WAVE_32x64),
    (33 * 32, 512, 1032, WAVE_64x64), (1, 5120, 1280, WAVE_32x32), (31, 72, 264, WAVE_32x32),
    # a 96 x 64 workgroup has a CU to itself: one round of them at most
    (1536, 1024, 1024, WAVE_96x64), (1537, 1024, 1024, WAVE_64x64), (1025, 3632, 1360, WAVE_64x64),
    # of 32 x 64 a CU holds several
    (128, 4096, 1544, WAVE_32x64), (32, 30592, 512, WAVE_32x64)])
def test_tile_of_few_rows(M, N, K, kernel, b_t):
    assert choice(M, N, K, b_t=b_t) == kernel


@pytest.mark.parametrize("M, N, K, epilogue, a_t", [(1536, 768, 1024, hn.EPI_NONE, False), (64, 64, 64, hn.EPI_BIAS, False), (4096, 4096, 1024, hn.EPI_BIAS_GELU, False),
                                                    (1024, 1024, 512, hn.EPI_ACCUM_F32, True), (4096, 4096, 4096, hn.EPI_ACCUM_F32, True)])
def test_rows_of_the_output_may_be_any_distance_apart(M, N, K, epilogue, a_t):
    for dtype in (hn.BF16, hn.FP32):
        near = choice(M, N, K, epilogue=epilogue, a_t=a_t, dtype=dtype)
        assert near != ALU
        for ldc in (2 ** 28 - 4, 2 ** 28, 2 ** 31 - 4):
            assert choice(M, N, K, ldc=ldc, epilogue=epilogue, a_t=a_t, dtype=dtype) == near
