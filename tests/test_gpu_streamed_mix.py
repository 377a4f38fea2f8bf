"""GPU parity of steps whose verify items go along in the launch of the streamed chunk items: row blocks of eight and of four waves, in both orders
of the heads, narrow items, chains and trees, caches from none to several key ranges; and of one whose verify items are too many for that.  What the step
is meant to hold, that launch included, is asserted with the library's own planner."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import Pair, rel_err
from test_gpu_narrow_chunks import SHAPES, TOL

pytestmark = pytest.mark.gpu
MANY = {hd: dict(name="m%d" % hd, n_layers=1, d_model=h * hd, n_heads=h, head_dim=hd, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)
        for hd, h in ((64, 32), (128, 24))}
LIMITS = dict(max_devices=20, max_step_tokens=1664, max_pos=1664)
C, V = hi.CHUNK, hi.VERIFY
TREE = hi.tree_masks(hi.MEDUSA_LIKE_TREE)
# (models, segments of the step, what it holds: streamed row blocks, waves of a block, narrow items, verify items, verify items along, heads in turn)
CASES = {
    "eight waves": (SHAPES, [(0, C, 70, 40), (1, V, 0, 1), (2, V, 33, 8, TREE), (3, C, 300, 64), (4, V, 1100, 5), (5, V, 47, 3)], (4, 8, 0, 8, True, True)),
    "four waves": (MANY, [(0, C, 40, 300), (1, V, 15, 8, TREE), (2, C, 0, 200), (3, V, 600, 5)], (17, 4, 0, 4, True, True)),
    # more than 256 blocks x heads of unequal lengths over 800 keys: a block in all heads of an XCD before the next
    "heads together": (MANY, [(0, C, 900, 200), (1, V, 1000, 5), (2, C, 300, 100), (3, C, 1200, 70), (4, V, 33, 8, TREE)], (14, 4, 0, 5, True, False)),
    "narrow": (SHAPES, [(0, C, 33, 20), (1, V, 31, 2), (2, C, 700, 32), (3, V, 1000, 8, TREE), (4, C, 0, 1), (5, V, 0, 8)], (0, 0, 4, 6, True, True)),
    "blocks and narrow": (SHAPES, [(0, C, 1540, 17), (1, C, 100, 90), (2, V, 640, 4), (3, V, 5, 8, TREE)], (3, 8, 5, 4, True, True)),
    # eight waves and more than 256 verify items x heads: a launch of their own
    "too many for eight waves": (MANY, [(0, C, 300, 64)] + [(i, V, 100 + 7 * i, 5) for i in range(1, 13)], (2, 8, 0, 12, False, True)),
}


def plan(cfg, segs):
    from paper_2503_18989_amd import HatPlanner
    p = HatPlanner(cfg, 800, **LIMITS)
    for sg in segs:
        if sg[2]:
            p.plan([(sg[0], C, 0, sg[2])])
    q = p.plan(segs)
    blocks = p.blocks()
    keys = [min(b["kv_end"], b["start"] + b["q0"] + b["nq"]) - b["kv_begin"] for b in blocks]
    together = cfg["n_heads"] % 8 == 0 and len(keys) * cfg["n_heads"] > 256 and max(keys) >= 800 and max(keys) * len(keys) > 1.1 * sum(keys)
    got = len(blocks), p.block_waves(), p.narrow_items(), len(q["verify_items"]), p.verify_along(), not together
    p.close()
    return got


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("name", list(CASES))
def test_verify_items_in_the_launch_of_the_chunk_items(name, hd, kv):
    models, segs, holds = CASES[name]
    cfg = models[hd]
    assert plan(cfg, segs) == holds
    p = Pair(cfg, 79, n_pages=800, kv_dtype=kv, **LIMITS)
    for sg in segs:
        if sg[2]:
            p.step([(sg[0], C, 0, sg[2])])
    for sg, o, r in zip(segs, *p.step(segs)):
        assert np.all(np.isfinite(o)) and rel_err(o, r) <= TOL, (sg[:4], rel_err(o, r))
    p.check_pages(range(len(segs)))
    p.close()
