"""LayerNorm gradients are added up beside the weight gradients' tiles or in a launch of their own: the same bits."""

import numpy as np
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


def in_order(rows):
    """The sum over axis 0 as every kernel adds it: 32 groups each take every 32nd row, then the groups in order."""
    groups = np.zeros((32,) + rows.shape[1:], np.float32)
    for r, row in enumerate(rows):
        groups[r % 32] += row
    total = np.zeros(rows.shape[1:], np.float32)
    for g in groups:
        total += g
    return total


# the kernel whose wavefronts split the contraction (0, 1, and what the sizes choose), which takes the sums along in both types, and the
# others; the partial rows are read from the end of the workspace, 256 rows for each LayerNorm, in the order of the backward pass
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("config", [-1, 0, 1, 7, 9, 10])
@pytest.mark.parametrize("norm, hidden, seq, mb, blocks", [("pre", 256, 128, 1, 1), ("post", 288, 33, 2, 2), ("pre", 648, 777, 1, 2), ("post", 1024, 1100, 4, 1)])
def test_layernorm_gradients_are_the_partial_rows_in_order(norm, hidden, seq, mb, blocks, config, dtype):
    import torch
    from paper_2308_15762_amd import hanayo as hn

    kind, esz = (torch.bfloat16, 2) if dtype == "bf16" else (torch.float32, 4)
    g = torch.Generator(device="cuda").manual_seed(hidden + seq)
    desc = hn.make_desc(blocks, hidden, hidden // 8 if hidden % 32 else hidden // 32, 4 * hidden, seq, mb, hn.PRE_LN if norm == "pre" else hn.POST_LN,
                        hn.MASK_CAUSAL if norm == "pre" else hn.MASK_NONE, hn.BF16 if dtype == "bf16" else hn.FP32)
    draw = lambda n, std: torch.empty(n, dtype=kind, device="cuda").normal_(0, std, generator=g)  # noqa: E731
    room = lambda n: torch.zeros(int(n), dtype=torch.uint8, device="cuda")  # noqa: E731
    w = draw(hn.hanayo_weight_bytes(desc) // esz, 0.02)
    x, dy = (draw(mb * seq * hidden, 1.0) for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    stash, work = room(hn.hanayo_stash_bytes(desc)), room(hn.hanayo_workspace_bytes(desc))
    grads = torch.zeros(hn.hanayo_grad_bytes(desc) // 4, device="cuda")
    hn.hanayo_op_gemm_config(config)
    try:
        hn.hanayo_chunk_forward(desc, w, x, None, y, stash, work)
        for _ in range(2):   # the sums are added to what is there
            hn.hanayo_chunk_backward(desc, w, grads, dy, None, stash, dx, work)
    finally:
        hn.hanayo_op_gemm_config(-1)
    slots = work[-2 * blocks * 256 * 2 * hidden * 4:].view(torch.float32).view(2 * blocks, 256, 2 * hidden).cpu().numpy()
    per_workgroup = 16 // ((hidden + 511) // 512)
    written = min(256, -(-mb * seq // per_workgroup))
    for at, (b, ln) in enumerate((b, ln) for b in range(blocks)[::-1] for ln in ("ln2", "ln1")):
        want = in_order(slots[at, :written])
        for name, half in ((ln + "_g", want[:hidden]), (ln + "_b", want[hidden:])):
            first, count = hn.hanayo_param_span(desc, b, hn.PARAM_NAMES.index(name))
            got = grads[first:first + count].cpu().numpy()
            assert np.abs(half).max() > 0 and (got == half + half).all(), (b, name)
