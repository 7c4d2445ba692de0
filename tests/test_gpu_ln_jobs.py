"""LayerNorm gradients are added up beside the weight gradients' tiles or in a launch of their own: the same bits."""

import pytest

pytestmark = pytest.mark.gpu


# tile configurations 9 and 10 take the sums along, 7 leaves them to one launch for all blocks
@pytest.mark.parametrize("hidden, seq, mb, blocks", [(256, 128, 1, 1), (288, 33, 2, 2), (640, 777, 1, 2), (1024, 300, 1, 3)])
@pytest.mark.parametrize("norm", ["pre", "post"])
def test_layernorm_gradients_do_not_depend_on_the_launch(norm, hidden, seq, mb, blocks):
    import torch
    from paper_2308_15762_amd import hanayo as hn

    g = torch.Generator(device="cuda").manual_seed(hidden + seq)
    desc = hn.make_desc(blocks, hidden, hidden // 32, 4 * hidden, seq, mb, hn.PRE_LN if norm == "pre" else hn.POST_LN,
                        hn.MASK_CAUSAL if norm == "pre" else hn.MASK_NONE, hn.BF16)
    draw = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)  # noqa: E731
    room = lambda n: torch.zeros(int(n), dtype=torch.uint8, device="cuda")  # noqa: E731
    w = draw(hn.hanayo_weight_bytes(desc) // 2, 0.02)
    x, dy = (draw(mb * seq * hidden, 1.0) for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    stash, work = room(hn.hanayo_stash_bytes(desc)), room(hn.hanayo_workspace_bytes(desc))
    got = []
    try:
        for config in (7, 9, 10):
            hn.hanayo_op_gemm_config(config)
            grads = torch.zeros(hn.hanayo_grad_bytes(desc) // 4, device="cuda")
            hn.hanayo_chunk_forward(desc, w, x, None, y, stash, work)
            for _ in range(2):   # the sums are added to what is there
                hn.hanayo_chunk_backward(desc, w, grads, dy, None, stash, dx, work)
            got.append(grads)
    finally:
        hn.hanayo_op_gemm_config(-1)
    for b in range(blocks):
        for i, name in enumerate(hn.PARAM_NAMES):
            if name.startswith("ln"):
                at, count = hn.hanayo_param_span(desc, b, i)
                first = got[0][at:at + count]
                assert first.abs().max() > 0
                for other in got[1:]:
                    assert torch.equal(first, other[at:at + count]), (b, name)
