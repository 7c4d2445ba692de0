"""The tiles of the kernel whose wavefronts split the contraction give the same bits: 96 x 64 and 32 x 64, which the automatic
choice takes where they need fewer rounds of the CUs, against 64 x 64 (gemm config 0), in and at the edges of their ranges."""

import pytest
import torch

from paper_2308_15762_amd import hanayo as hn

pytestmark = pytest.mark.gpu

LAYOUTS = {"fwd": ([hn.EPI_NONE, hn.EPI_BIAS, hn.EPI_BIAS_GELU, hn.EPI_BIAS_RES], True), "dx": ([hn.EPI_NONE, hn.EPI_MUL_DGELU, hn.EPI_ADD], False)}


# (test_host_gemm_choice.py holds which tile these go to.)  96 x 64: 192 tiles, whole and ragged, one row into the last tile, K below
# and past a K tile, 256 tiles and one tile row more (square again); 32 x 64: 250 tiles, N ending inside a tile, 256, few rows, 478 (the
# instance with one stage); 264 tiles of 32 x 64 would be 64 x 64; 64 and less: the square tiles
@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("M, N, K", [(1536, 768, 1024), (1527, 768, 3072), (1441, 760, 2056), (700, 1536, 1608), (777, 640, 2560), (769, 632, 520),
                                     (1024, 512, 2048), (33 * 32, 512, 1032), (96, 3840, 1288), (1, 5120, 1280), (31, 72, 264),
                                     (1536, 1024, 1024), (1537, 1024, 1024), (1025, 3632, 1360), (128, 4096, 1544), (32, 30592, 512)])
def test_tiles_give_the_same_bits(layout, M, N, K):
    epis, b_t = LAYOUTS[layout]
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    draw = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    A, B, bias, aux = draw(M, K), draw(*((K, N) if b_t else (N, K))), draw(N), draw(M, N)
    for epi in epis:
        got = []
        try:
            for config in (0, 1, -1):
                hn.hanayo_op_gemm_config(config)
                C, pre = torch.full_like(aux, 7.0), torch.full_like(aux, 7.0)
                hn.hanayo_op_gemm(hn.BF16, A, B, C, M, N, K, K, N if b_t else K, N, False, b_t, epi, bias, aux, pre)
                got.append((C, pre))
        finally:
            hn.hanayo_op_gemm_config(-1)
        exact = A.float() @ (B if b_t else B.T).float()
        if epi == hn.EPI_NONE:
            assert (got[0][0].float() - exact).norm() <= 3e-3 * exact.norm()   # bf16 storage: 2^-9 of every element
        for other in got[1:]:
            assert torch.equal(got[0][0], other[0]) and torch.equal(got[0][1], other[1]), epi


def strided(rows, cols, ld, values):
    """`values` in rows `ld` elements apart."""
    room = torch.empty((rows - 1) * ld + cols, dtype=torch.bfloat16, device="cuda")
    view = torch.as_strided(room, (rows, cols), (ld, 1))
    view.copy_(values)
    return room, view


# the last stride whose 96 rows a lane's offset reaches, the first that it does not (64-row tiles take it), the last for 64 rows
@pytest.mark.parametrize("lda", [(2 ** 31 - 1) // 192 // 8 * 8, (2 ** 31 - 1) // 192 // 8 * 8 + 8, (2 ** 31 - 1) // 128 // 8 * 8])
def test_rows_far_apart(lda):
    M, N, K = 200, 5000, 1024
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    A, B, want, got = draw(M, K), draw(K, N), draw(M, N), draw(M, N)
    wide, _ = strided(M, K, lda, A)
    hn.hanayo_op_gemm(hn.BF16, A, B, want, M, N, K, K, N, N, False, True, hn.EPI_NONE)
    hn.hanayo_op_gemm(hn.BF16, wide, B, got, M, N, K, lda, N, N, False, True, hn.EPI_NONE)
    assert torch.equal(want, got)


# 2^28 elements between rows of C and beyond, on both kinds of kernel (9: 128 x 128 tiles loaded straight into LDS)
@pytest.mark.parametrize("config", [0, 9])
@pytest.mark.parametrize("ldc, M", [(2 ** 28, 5), (2 ** 28 + 4, 5), (2 ** 31 - 4, 2)])
def test_rows_of_the_output_far_apart(ldc, M, config):
    N, K = 136, 264
    g = torch.Generator(device="cuda").manual_seed(6)
    draw = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    A, B, want = draw(M, K), draw(K, N), draw(M, N)
    room, view = strided(M, N, ldc, draw(M, N))
    hn.hanayo_op_gemm_config(config)
    try:
        hn.hanayo_op_gemm(hn.BF16, A, B, want, M, N, K, K, N, N, False, True, hn.EPI_NONE)
        hn.hanayo_op_gemm(hn.BF16, A, B, room, M, N, K, K, N, ldc, False, True, hn.EPI_NONE)
    finally:
        hn.hanayo_op_gemm_config(-1)
    assert torch.equal(want, view)
