"""GPU parity of chunk items of more than 32 rows on both of their ways: streamed in blocks of 32 rows, and staged through LDS (a
workgroup target other than the default).  That a step takes the way it is meant to is asserted with the library's own planner."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import Pair, rel_err
from test_gpu_narrow_chunks import SHAPES, TOL

pytestmark = pytest.mark.gpu


def planned_blocks(cfg, segs, target=256):
    """(row blocks, waves of each) with which the library streams a step of (start, rows), one device each; (0, 0): staged"""
    from paper_2503_18989_amd import HatPlanner
    p = HatPlanner(cfg, 800, max_devices=len(segs), max_step_tokens=1664, max_pos=1664)
    p.set_attn_targets(target, 2048)
    for d, (s, _) in enumerate(segs):
        if s:
            p.plan([(d, hi.CHUNK, 0, s)])
    p.plan([(d, hi.CHUNK, s, n) for d, (s, n) in enumerate(segs)])
    r = len(p.blocks()), p.block_waves()
    p.close()
    return r


# rows at the edges of a block and of an item, over no keys, a few, and enough for key ranges (from about 1000 keys on)
CASES = [([33, 64, 65, 96], [0, 15, 700, 1500]), ([255, 256, 257], [1290, 1, 47]), ([300, 40, 7, 128], [500, 1040, 33, 0])]


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
def test_streamed_and_staged_chunks_against_the_oracle(hd, kv):
    for rows, starts in CASES:
        for target in (256, 4096, 64):        # streamed; staged in as many key ranges as fit; staged with the keys whole
            assert (planned_blocks(SHAPES[hd], list(zip(starts, rows)), target)[0] > 0) == (target == 256)
            p = Pair(SHAPES[hd], 78, n_pages=4 * 104, max_devices=4, max_step_tokens=1600, max_pos=1664, kv_dtype=kv)
            p.gpu.set_attn_targets(target, 2048)
            for d, s in enumerate(starts):
                if s:
                    p.step([(d, hi.CHUNK, 0, s)])
            for o, r in zip(*p.step([(d, hi.CHUNK, s, n) for d, (s, n) in enumerate(zip(starts, rows))])):
                assert np.all(np.isfinite(o)) and rel_err(o, r) <= TOL, (rows, target, rel_err(o, r))
            p.check_pages(range(len(rows)))
            p.close()


def test_many_workgroups_of_both_sizes():
    # attention output against float64 softmax over the same queries and cache rows: probabilities and output are each rounded to
    # fp16, sqrt(2) * 2^-11.5 of a row's size in all; bounded by 2^-10 (a bf16 cache: an fp16 one is exported rounded to bf16).  7B-shaped heads: 224 workgroups
    # of eight waves, 672 of four (head by head; with a block of 964 keys the heads of an XCD together) and 416 of eight in two rounds.
    import torch
    from gpu_util import dev_weights
    from paper_2503_18989_amd import HatMid, Segment
    cfg = dict(name="s7", n_layers=1, d_model=4096, n_heads=32, head_dim=128, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)
    d, H, hd = 4096, 32, 128
    gen = torch.Generator(device="cuda").manual_seed(6)
    w = {k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
         for k, s in dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(512, d), w_up=(512, d), w_down=(d, 512)).items()}
    m = HatMid(cfg, [w], n_pages=200, max_devices=4, max_step_tokens=1024, max_pos=1088, io_dtype="f32")
    for segs, want in (([(100, 200)], (7, 8)), ([(300, 130), (170, 64)], (7, 8)), ([(0, 333), (401, 256), (90, 50)], (21, 4)),
                       ([(900, 64), (100, 333), (401, 256)], (21, 4)), ([(950, 70), (90, 60), (500, 100), (200, 120)], (13, 8))):
        assert planned_blocks(cfg, segs) == want, segs
        for dev, (s, _) in enumerate(segs):
            if s:
                k, v = (torch.randn((s, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2))
                m.kv_import(dev, 0, 0, k, v)
        m.forward([Segment(dev, hi.CHUNK, s, torch.randn((n, d), device="cuda", generator=gen)) for dev, (s, n) in enumerate(segs)])
        T = sum(n for _, n in segs)
        q, o = (m.debug_dump(x, T).double().view(T, H, hd) for x in ("q", "attn"))
        t = 0
        for dev, (s, n) in enumerate(segs):
            K, V = (x.double() for x in m.kv_export(dev, 0, 0, s + n))
            hidden = torch.arange(s + n, device="cuda")[None, :] > s + torch.arange(n, device="cuda")[:, None]
            for h in range(H):
                p = torch.softmax(((q[t:t + n, h] @ K[:, h].T.contiguous()) / hd ** 0.5).masked_fill(hidden, -float("inf")), -1)
                ref = p @ V[:, h].contiguous()
                assert float((o[t:t + n, h] - ref).norm() / ref.norm()) <= 2.0 ** -10, (segs, dev, h)
            t += n
    m.close()
