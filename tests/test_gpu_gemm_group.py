"""Groups of products of any layout and epilogue: one launch, and the results of one product at a time."""

import ctypes

import pytest
import torch

from paper_2308_15762_amd import hanayo as hn

pytestmark = pytest.mark.gpu

CASES = [(b_t, epi) for b_t, epis in ((True, (hn.EPI_NONE, hn.EPI_BIAS, hn.EPI_BIAS_GELU, hn.EPI_BIAS_RES)), (False, (hn.EPI_NONE, hn.EPI_MUL_DGELU, hn.EPI_ADD)))
         for epi in epis]


def problems(dtype, shapes, b_t):
    kind = torch.bfloat16 if dtype == hn.BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(len(shapes))
    draw = lambda *s: torch.empty(s, dtype=kind, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    return [dict(A=draw(M, K), B=draw(K, N) if b_t else draw(N, K), C=draw(M, N), bias=draw(N), aux=draw(M, N), aux_out=draw(M, N), M=M, N=N, K=K,
                 lda=K, ldb=N if b_t else K, ldc=N) for M, N, K in shapes]


def launches(call):
    """How many kernels `call(stream)` enqueues: the nodes of a graph captured from it."""
    call(None)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call(torch.cuda.current_stream().cuda_stream)
    count = ctypes.c_size_t()
    assert hn._lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# 0: 64 x 64 tiles over split wavefronts, 1: 32 x 32, 7, 9 - 11: tiles loaded straight into LDS
@pytest.mark.parametrize("dtype, config", [(hn.BF16, c) for c in (-1, 0, 1, 7, 9, 10, 11)] + [(hn.FP32, c) for c in (-1, 0, 1)])
@pytest.mark.parametrize("shapes", [[(512, 512, 512)] * 4, [(256, 256, 128)] * 2, [(777, 640, 264), (8, 72, 1032), (300, 8, 64)], [(31, 136, 200)]])
def test_a_group_is_one_launch_with_the_results_of_single_products(shapes, dtype, config):
    hn.hanayo_op_gemm_config(config)
    try:
        for b_t, epi in CASES:
            group = problems(dtype, shapes, b_t)
            one = launches(lambda stream: hn.hanayo_op_gemm_group(dtype, False, b_t, epi, group, stream=stream))
            assert one == 1, (b_t, epi)
            hn.hanayo_op_gemm_group(dtype, False, b_t, epi, group)
            for p in group:
                want, pre = torch.empty_like(p["C"]), torch.zeros_like(p["C"])
                hn.hanayo_op_gemm(dtype, p["A"], p["B"], want, p["M"], p["N"], p["K"], p["lda"], p["ldb"], p["ldc"], False, b_t, epi, p["bias"], p["aux"], pre)
                if config != -1:   # the same kind of kernel, whose tiles all add in one order
                    assert torch.equal(p["C"], want), (b_t, epi)
                    assert epi != hn.EPI_BIAS_GELU or torch.equal(p["aux_out"], pre)
                else:              # two kinds may differ by the rounding of fp32 sums, in bf16 by one of the result
                    err = (p["C"].double() - want.double()).norm() / want.double().norm()
                    assert err <= (2.0 ** -8 if dtype == hn.BF16 else 1e-6 * p["K"] ** 0.5), (b_t, epi)
    finally:
        hn.hanayo_op_gemm_config(-1)
