"""GPU parity of steps whose verify items go along in the launch of the streamed chunk items: row blocks of eight and of four waves, narrow
items, chains and trees, caches from none to several key ranges.  What the step is meant to hold is asserted with the library's own planner."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import Pair, rel_err
from test_gpu_narrow_chunks import SHAPES, TOL

pytestmark = pytest.mark.gpu
MANY_HEADS = dict(name="n64x32", n_layers=1, d_model=2048, n_heads=32, head_dim=64, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)
C, V = hi.CHUNK, hi.VERIFY
TREE = hi.tree_masks(hi.MEDUSA_LIKE_TREE)
# (model, segments of the step, streamed row blocks expected, waves of a block, narrow items expected)
CASES = {
    "eight waves": ("both", [(0, C, 70, 40), (1, V, 0, 1), (2, V, 33, 8, TREE), (3, C, 300, 64), (4, V, 1100, 5), (5, V, 47, 3)], True, 8, 0),
    "four waves": (MANY_HEADS, [(0, C, 40, 300), (1, V, 15, 8, TREE), (2, C, 0, 129), (3, V, 600, 5)], True, 4, 0),
    "narrow": ("both", [(0, C, 33, 20), (1, V, 31, 2), (2, C, 700, 32), (3, V, 1000, 8, TREE), (4, C, 0, 1), (5, V, 0, 8)], False, 0, 6),
    "blocks and narrow": ("both", [(0, C, 1540, 17), (1, C, 100, 90), (2, V, 640, 4), (3, V, 5, 8, TREE)], True, 8, 2),
}


def plan(cfg, segs):
    from paper_2503_18989_amd import HatPlanner
    p = HatPlanner(cfg, 800, max_devices=8, max_step_tokens=1664, max_pos=1664)
    for sg in segs:
        if sg[2]:
            p.plan([(sg[0], C, 0, sg[2])])
    p.plan(segs)
    r = len(p.blocks()), p.block_waves(), p.narrow_items()
    p.close()
    return r


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("name", list(CASES))
def test_verify_items_in_the_launch_of_the_chunk_items(name, hd, kv):
    model, segs, blocks, waves, narrow = CASES[name]
    if model != "both" and hd == 128:
        pytest.skip("one model")
    cfg = SHAPES[hd] if model == "both" else model
    got = plan(cfg, segs)
    assert ((got[0] > 0), got[1]) == (blocks, waves) and (got[2] > 0) == (narrow > 0), got
    p = Pair(cfg, 79, n_pages=800, max_devices=8, max_step_tokens=1664, max_pos=1664, kv_dtype=kv)
    for sg in segs:
        if sg[2]:
            p.step([(sg[0], C, 0, sg[2])])
    for sg, o, r in zip(segs, *p.step(segs)):
        assert np.all(np.isfinite(o)) and rel_err(o, r) <= TOL, (sg[:4], rel_err(o, r))
    p.check_pages(range(len(segs)))
    p.close()
