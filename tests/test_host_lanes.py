"""How many of its lanes the executor uses, by the size of a chunk's products (no GPU)."""

import pytest

from paper_2308_15762_amd import hanayo as hn


@pytest.mark.parametrize("tokens, ffn, most", [
    (4096, 4096, 4),          # 16 x 16 tiles of 256 x 256
    (4096 - 256, 4096, 2),    # 15 x 16
    (4096 - 255, 4096, 4),    # 15 whole tile rows and one more row
    (128, 1024, 2),
    (2048, 10240, 4),
])
def test_small_tasks_use_two_lanes(tokens, ffn, most):
    tasks = hn.hanayo_schedule(4, 2, 8, 0)
    desc = hn.make_desc(1, 256, 4, ffn, tokens, 1, hn.PRE_LN, hn.MASK_CAUSAL, hn.BF16)
    for lanes in (1, 2, 3, 4):
        lane, deps = hn.hanayo_executor_plan(tasks, 4, 2, 8, 0, lanes, desc)
        want, want_deps = hn.hanayo_executor_plan(tasks, 4, 2, 8, 0, min(lanes, most))
        assert (lane == want).all() and (deps == want_deps).all()
        assert len(set(lane.tolist())) == min(lanes, most)
