"""bf16 attention backward: a masked (query, key) pair has probability zero whatever the query's log-sum-exp holds (NaN, minus infinity),
so that alone reaches no gradient of the keys that the mask keeps from the query.  (An output or output gradient that is not
finite still does, as zero times NaN in dK; and at head dim 64 the 128-row kernels mask the scores before the exponential.)"""

import pytest
import torch

from paper_2308_15762_amd import hanayo as hn

pytestmark = pytest.mark.gpu


def backward(qkv, vl, ctx, lse, dctx, b, s, heads, d, causal):
    dqkv, delta = torch.full_like(qkv, 7.0), torch.empty_like(lse)
    hn.hanayo_op_attention_backward(hn.BF16, qkv, vl, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal)
    torch.cuda.synchronize()
    return dqkv.view(b, s, 3, heads * d).clone()


# few rows (32-row workgroups) and many (128-row ones) for every head dim that is loaded straight into LDS; 40 and 72 are not
@pytest.mark.parametrize("bad", [float("nan"), float("-inf")])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("b,s,heads,d", [(2, 100, 2, 32), (2, 150, 2, 64), (1, 140, 3, 80), (2, 97, 2, 96), (1, 161, 2, 128), (1, 90, 2, 40), (1, 90, 2, 72),
                                         (7, 130, 16, 32), (2, 250, 33, 80), (2, 300, 40, 96), (2, 130, 40, 128)])
def test_bad_log_sum_exp_stays_before_the_mask(b, s, heads, d, causal, bad):
    g = torch.Generator(device="cuda").manual_seed(s + d)
    draw = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    qkv, dctx = draw(b, s, 3 * heads * d), draw(b, s, heads * d)
    vl = None if causal else torch.full((b,), s - 45, dtype=torch.int32, device="cuda")
    ctx, lse = torch.empty_like(dctx), torch.empty((b, heads, s), device="cuda")
    hn.hanayo_op_attention_forward(hn.BF16, qkv, vl, ctx, lse, b, s, heads, d, causal)
    clean = backward(qkv, vl, ctx, lse, dctx, b, s, heads, d, causal)
    assert torch.isfinite(clean).all()
    row = 42   # inside a tile of queries; its tile mates' keys lie on both sides of the mask
    lse[0, :, row] = bad
    got = backward(qkv, vl, ctx, lse, dctx, b, s, heads, d, causal)
    assert not torch.isfinite(got[0, row, 0]).any()
    hidden = slice(row + 1, s) if causal else slice(s - 45, s)   # keys that query `row` does not see
    assert torch.equal(got[0, hidden, 1:], clean[0, hidden, 1:])
    assert torch.equal(got[1:], clean[1:])
