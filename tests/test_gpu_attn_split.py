"""bf16 attention at few rows (32-row workgroups whose wavefronts split the other side) and at head dim 32, against fp64.

Bound: probabilities, dS and stored results are rounded to bf16 (2^-9 relative each), and delta comes from a context rounded
the same way, so an output's error is at most 2^-8 of the sum of its absolute terms; with N(0, 1) operands that sum is
within four times the tensor's largest entry: 2^-6 of it."""

import numpy as np
import pytest
import torch

from paper_2308_15762_amd import hanayo as hn
from helpers import host
from test_gpu_attn_f32 import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,heads,d,causal,padded", [
    (1, 1, 1, 64, True, False), (1, 31, 3, 32, True, True), (2, 33, 2, 32, False, True), (1, 128, 2, 64, True, False),
    (1, 129, 8, 64, False, False), (2, 257, 4, 64, True, True), (1, 777, 2, 80, True, False), (2, 95, 3, 80, False, True),
    (1, 160, 2, 96, True, False), (1, 225, 1, 96, False, True), (1, 321, 2, 128, True, True), (2, 64, 8, 128, False, False),
    (3, 509, 16, 64, True, False), (2, 509, 16, 64, False, True),   # the last that split: 192 workgroups of 128 rows, 128
    (1, 385, 36, 64, False, False), (1, 481, 49, 32, True, False),  # backward only (144); none (196)
    (7, 130, 16, 32, True, True), (4, 261, 32, 32, False, True),    # head dim 32 in the 128-row kernels
    # both sides of the lines that depend on the sequence length
    (2, 250, 32, 64, True, False), (2, 250, 33, 64, True, False), (2, 250, 32, 80, True, False), (2, 250, 33, 80, True, False),
    (1, 256, 32, 128, False, True), (1, 256, 33, 128, False, True), (1, 300, 32, 96, False, False), (1, 300, 33, 96, False, False),
    (2, 128, 32, 128, True, False), (2, 128, 33, 128, True, False), (1, 770, 27, 80, True, False), (1, 770, 28, 80, True, False)])
def test_attention_bf16(b, s, heads, d, causal, padded):
    g = torch.Generator().manual_seed(s * 131 + d)
    H = heads * d
    qkv, dc = torch.randn((b, s, 3 * H), generator=g).bfloat16(), torch.randn((b, s, H), generator=g).bfloat16()
    vl = torch.randint(1, s + 1, (b,), generator=g, dtype=torch.int32) if padded else None
    ctx_ref, lse_ref, dqkv_ref = reference(qkv.float().numpy(), None if vl is None else vl.numpy(), dc.float().numpy(), heads, d, causal)
    qd, dcd, vd = qkv.cuda(), dc.cuda(), None if vl is None else vl.cuda()
    ctx, lse = torch.empty((b, s, H), dtype=torch.bfloat16, device="cuda"), torch.empty((b, heads, s), device="cuda")
    dqkv, delta = torch.full((b, s, 3 * H), 7.0, dtype=torch.bfloat16, device="cuda"), torch.empty((b, heads, s), device="cuda")
    hn.hanayo_op_attention_forward(hn.BF16, qd, vd, ctx, lse, b, s, heads, d, causal)
    hn.hanayo_op_attention_backward(hn.BF16, qd, vd, ctx, lse, dcd, dqkv, delta, b, s, heads, d, causal)
    torch.cuda.synchronize()
    assert np.abs(host(ctx) - ctx_ref).max() <= 2.0 ** -6 * np.abs(ctx_ref).max()
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 2.0 ** -12 * max(1.0, np.abs(lse_ref).max())
    for i, name in enumerate(("dq", "dk", "dv")):
        got, ref = host(dqkv)[..., i * H:(i + 1) * H], dqkv_ref[..., i * H:(i + 1) * H]
        assert np.abs(got - ref).max() <= 2.0 ** -6 * max(np.abs(ref).max(), 1.0), name
