"""The GEMM kernels at the edges of their tiles and of their K tile, against fp64: the one that splits the contraction over
a workgroup's wavefronts (gemm config 0: 64 x 64 tiles, 1: 32 x 32) and the direct-to-LDS kernels (7, 9, 10, 11; bf16 only).

Bound: a sum of K products in fp32 is off by at most (K + 4) 2^-24 sum |a b|, whatever its order; the fp32 epilogue
(bias, residual, GELU) adds a few roundings of the result, and bf16 storage 2^-8 of it."""

import numpy as np
import pytest
import torch

from oracle import block as OB
from paper_2308_15762_amd import hanayo as hn
from paper_2308_15762_amd import synth
from helpers import dev, host

pytestmark = pytest.mark.gpu

LAYOUTS = {"fwd": (False, True), "dx": (False, False), "dw": (True, True)}
EPIS = {"fwd": [hn.EPI_BIAS, hn.EPI_BIAS_GELU, hn.EPI_BIAS_RES], "dx": [hn.EPI_NONE, hn.EPI_MUL_DGELU, hn.EPI_ADD], "dw": [hn.EPI_ACCUM_F32]}


# every kernel with the types it takes
KERNELS = [(c, "bf16") for c in (0, 1, 7, 9, 10, 11)] + [(0, "fp32"), (1, "fp32")]


@pytest.fixture(params=KERNELS, ids=lambda k: "%d-%s" % k)
def kernel(request):
    hn.hanayo_op_gemm_config(request.param[0])
    yield request.param
    hn.hanayo_op_gemm_config(-1)


# (M, N, K): M is ragged for fwd and dx, K (the tokens) for dw; the rest are multiples of 8
@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (63, 64, 64), (65, 72, 136), (129, 56, 320), (64, 128, 1024), (777, 104, 264), (333, 520, 96), (513, 264, 200), (256, 384, 72)])
def test_gemm_edges(kernel, layout, M, N, K):
    dtype = kernel[1]
    if layout == "dw":
        M, N, K = K, N, M
    a_t, b_t = LAYOUTS[layout]
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    rnd = lambda *s: synth.bf16_round(rng.normal(size=s)) if dtype == "bf16" else rng.normal(size=s).astype(np.float32)
    A, B, bias, aux = rnd(M, K), rnd(K, N), rnd(N), rnd(M, N)
    ref = A.astype(np.float64) @ B
    sums = np.abs(A).astype(np.float64) @ np.abs(B)
    Ad, Bd = dev(A.T.copy() if a_t else A, dtype), dev(B if b_t else B.T.copy(), dtype)
    for epi in EPIS[layout]:
        gain = 1.0                              # what the epilogue multiplies the product's error by
        if epi == hn.EPI_ACCUM_F32:
            C = torch.from_numpy(aux.astype(np.float32)).cuda()
            want = aux + ref
        else:
            C = torch.empty((M, N), dtype=Ad.dtype, device="cuda")
            if epi == hn.EPI_MUL_DGELU:
                gain = 1.2                      # |GELU'| < 1.13
            want = {hn.EPI_NONE: ref, hn.EPI_BIAS: ref + bias, hn.EPI_BIAS_GELU: OB.gelu(ref + bias), hn.EPI_BIAS_RES: ref + bias + aux,
                    hn.EPI_MUL_DGELU: ref * OB.gelu_grad(aux.astype(np.float64)), hn.EPI_ADD: ref + aux}[epi]
            gain = 1.2 if epi == hn.EPI_BIAS_GELU else gain
        pre = torch.empty((M, N), dtype=Ad.dtype, device="cuda")
        cs = torch.zeros(N, dtype=torch.float32, device="cuda") if epi == hn.EPI_ACCUM_F32 else None
        scratch = torch.empty(64 * N, dtype=torch.float32, device="cuda") if cs is not None else None
        hn.hanayo_op_gemm(hn.BF16 if dtype == "bf16" else hn.FP32, Ad, Bd, C, M, N, K, M if a_t else K, N if b_t else K, N, a_t, b_t, epi,
                          dev(bias, dtype), dev(aux, dtype), pre, cs, scratch)
        torch.cuda.synchronize()
        store = 2.0 ** -8 if dtype == "bf16" and epi != hn.EPI_ACCUM_F32 else 0.0
        bound = (K + 4) * 2.0 ** -24 * gain * sums + (store + 2.0 ** -20) * (np.abs(want) + np.abs(ref) + 1.0)
        assert (np.abs(host(C) - want) <= bound).all(), "epilogue %d" % epi
        if epi == hn.EPI_BIAS_GELU:
            assert (np.abs(host(pre) - (ref + bias)) <= bound + (store + 2.0 ** -20) * np.abs(ref + bias)).all()
        if cs is not None:
            assert (np.abs(cs.cpu().numpy() - B.astype(np.float64).sum(0)) <= (K + 4) * 2.0 ** -24 * np.abs(B).sum(0) + 1e-30).all()


def test_gemm_group_edges(kernel):
    """Four weight gradients of different sizes and an odd token count in one launch."""
    dtype = kernel[1]
    rng = np.random.default_rng(5)
    K, probs, want = 201, [], []
    for M, N in [(72, 136), (136, 72), (8, 264), (200, 8)]:
        A, B = (synth.bf16_round(rng.normal(size=(K, n))) for n in (M, N))
        probs.append(dict(A=dev(A, dtype), B=dev(B, dtype), C=torch.ones((M, N), device="cuda"), M=M, N=N, K=K, lda=M, ldb=N, ldc=N,
                          colsum=torch.zeros(N, device="cuda"), colsum_scratch=torch.empty(64 * N, device="cuda")))
        want.append((1.0 + A.astype(np.float64).T @ B, np.abs(A).astype(np.float64).T @ np.abs(B), B.astype(np.float64).sum(0), np.abs(B).sum(0)))
    hn.hanayo_op_gemm_group(hn.BF16 if dtype == "bf16" else hn.FP32, True, True, hn.EPI_ACCUM_F32, probs)
    torch.cuda.synchronize()
    for p, (c, ca, s, sa) in zip(probs, want):
        assert (np.abs(p["C"].cpu().numpy() - c) <= (K + 4) * 2.0 ** -24 * (ca + 1.0)).all()
        assert (np.abs(p["colsum"].cpu().numpy() - s) <= (K + 4) * 2.0 ** -24 * sa).all()


def placed(a, pitch, dtype, shift=0, fill=float("nan")):
    """`a` on the device with row pitch `pitch`, its first element `shift` elements behind an aligned address; the gaps hold `fill`."""
    rows, cols = a.shape
    flat = torch.full((shift + rows * pitch,), fill, device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    t = flat[shift:].view(rows, pitch)
    t[:, :cols] = dev(np.ascontiguousarray(a), dtype)
    return t


def check_gemm(dtype, layout, epi, M, N, K, pads=(0, 0, 0), shifts=(0, 0, 0)):
    """One product with pitches pads = (A, B, C) wider than the rows and bases off by shifts elements, against fp64."""
    a_t, b_t = LAYOUTS[layout]
    rng = np.random.default_rng(M * 5 + N * 3 + K + epi)
    rnd = lambda *s: synth.bf16_round(rng.normal(size=s)) if dtype == "bf16" else rng.normal(size=s).astype(np.float32)
    A, B, bias, aux = rnd(M, K), rnd(K, N), rnd(N), rnd(M, N)
    ref, sums = A.astype(np.float64) @ B, np.abs(A).astype(np.float64) @ np.abs(B)
    want = {hn.EPI_NONE: ref, hn.EPI_BIAS: ref + bias, hn.EPI_BIAS_GELU: OB.gelu(ref + bias), hn.EPI_BIAS_RES: ref + bias + aux,
            hn.EPI_MUL_DGELU: ref * OB.gelu_grad(aux.astype(np.float64)), hn.EPI_ADD: ref + aux, hn.EPI_ACCUM_F32: ref + aux}[epi]
    lda, ldb, ldc = (M if a_t else K) + pads[0], (N if b_t else K) + pads[1], N + pads[2]
    Ad, Bd = placed(A.T if a_t else A, lda, dtype, shifts[0]), placed(B if b_t else B.T, ldb, dtype, shifts[1])
    cdt = "fp32" if epi == hn.EPI_ACCUM_F32 else dtype
    C = placed(aux if epi == hn.EPI_ACCUM_F32 else 0 * aux, ldc, cdt, shifts[2], 7.0)
    auxd, pre = placed(aux, ldc, dtype, shifts[2]), placed(0 * aux, ldc, dtype, shifts[2], 7.0)
    hn.hanayo_op_gemm(hn.BF16 if dtype == "bf16" else hn.FP32, Ad, Bd, C, M, N, K, lda, ldb, ldc, a_t, b_t, epi, dev(bias, dtype), auxd, pre)
    torch.cuda.synchronize()
    store = 2.0 ** -8 if cdt == "bf16" else 0.0
    bound = (K + 4) * 2.0 ** -24 * 1.2 * sums + (store + 2.0 ** -20) * (np.abs(want) + np.abs(ref) + 1.0)
    assert (np.abs(host(C)[:, :N] - want) <= bound).all()
    if epi == hn.EPI_BIAS_GELU:
        assert (np.abs(host(pre)[:, :N] - (ref + bias)) <= bound + (store + 2.0 ** -20) * np.abs(ref + bias)).all()
    assert (host(C)[:, N:] == 7.0).all() and (host(pre)[:, N:] == 7.0).all()     # nothing past the rows


ALL = [(layout, epi) for layout in LAYOUTS for epi in EPIS[layout]]


@pytest.mark.parametrize("layout,epi", ALL)
@pytest.mark.parametrize("M,N,K,pads", [(256, 256, 128, (8, 16, 8)), (256, 256, 128, (0, 0, 4)), (72, 136, 96, (24, 8, 4))])
def test_gemm_pitches(kernel, layout, epi, M, N, K, pads):
    """Leading dimensions wider than the rows, also where those of C start on 8-byte boundaries only (bf16, ldc = 4 mod 8)."""
    check_gemm(kernel[1], layout, epi, M, N, K, pads)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("layout,epi", ALL)
@pytest.mark.parametrize("M,N,K,pads,shifts", [
    (65, 33, 47, (0, 0, 0), (0, 0, 0)), (64, 64, 64, (1, 2, 3), (0, 0, 0)),                                # no whole vectors, odd pitches
    (256, 256, 128, (0, 0, 0), (1, 0, 0)), (256, 256, 128, (0, 0, 0), (0, 2, 0)), (256, 256, 128, (0, 0, 0), (0, 0, 1))])   # bases off a boundary
def test_gemm_on_the_alu(dtype, layout, epi, M, N, K, pads, shifts):
    """What the matrix-instruction kernels do not take."""
    check_gemm(dtype, layout, epi, M, N, K, pads, shifts)


def test_gemm_on_the_alu_long_contraction():
    """More than 65536 contraction elements: the running sum is put aside every 65536."""
    check_gemm("fp32", "fwd", hn.EPI_NONE, 3, 5, 65536 + 65536 + 7)
