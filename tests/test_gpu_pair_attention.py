"""Chunks of at most 64 rows over an fp16 cache whose pages a small workgroup of their own reads, and the same chunks staged (a workgroup target
other than the default), against float64 softmax at the edges of row blocks, pages and stages.  Cache rows that nothing has written hold NaN.  That a step takes the
small workgroups is asserted with the library's own planner."""
import pytest

import hat_inputs as hi

CFG = dict(name="pairs", n_layers=1, d_model=4096, n_heads=32, head_dim=128, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)
LIMITS = dict(max_devices=24, max_step_tokens=1600, max_pos=1280)
# (first row, rows) of each device: caches that end on, before and behind a page and a stage of 32 keys
STEPS = {"lengths": [(896, 64), (897, 64), (911, 64), (912, 33), (960, 32), (1000, 63), (959, 64), (900, 1), (927, 34), (944, 48), (929, 47), (1001, 31)],
         "ends": [(900 + r, 45) for r in range(16)],        # on every row of a page
         "short": [(0, 64), (1, 63), (15, 64), (16, 33), (17, 64), (0, 40)] * 4}


def planned(segs, cfg=CFG, kv="f16", target=256):
    """(waves the planner reports, row blocks, chunk items) of the step"""
    from paper_2503_18989_amd import HatPlanner
    p = HatPlanner(cfg, 1600, kv_dtype=kv, **LIMITS)
    p.set_attn_targets(target, 2048)
    for sg in segs:
        if sg[1]:
            p.plan([(sg[0], hi.CHUNK, 0, sg[1])])
    items = p.plan([(d, k, s, n) for d, s, n, k in segs])["chunk_items"]
    r = p.block_waves(), len(p.blocks()), items
    p.close()
    return r


def chunks(step):
    return [(d, s, n, hi.CHUNK) for d, (s, n) in enumerate(step)]


@pytest.mark.parametrize("name", list(STEPS))
def test_steps_that_take_it(name):
    segs = chunks(STEPS[name])
    waves, blocks, items = planned(segs)
    assert (waves, blocks) == (2, 0) and len(items) == len(segs) and all(it["part_row"] < 0 for it in items)
    hd64 = dict(CFG, n_heads=64, head_dim=64)
    others = [planned(segs, kv="bf16"), planned(segs, cfg=hd64), planned(segs, target=255), planned(segs[:1]),           # other caches, heads, a wish, a small step,
              planned(segs[:-1] + [(len(segs) - 1, 900, 65, hi.CHUNK)]), planned(segs[:-1] + [(len(segs) - 1, 300, 5, hi.VERIFY)])]   # a longer chunk, a draft
    assert all(waves != 2 for waves, _, _ in others)


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(STEPS))
def test_chunks_that_read_their_pages_once(name):
    # probabilities, the staged way's partial results of key ranges and the output are rounded to fp16 once each: sqrt(3) * 2^-11.5 of a row's size in all.  The cached rows
    # are bf16 numbers; the step's own are exported rounded to bf16, 2^-9 of each.  Bounded by 2^-10 + 2^-9 for a device, by four times that for each row
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    step = STEPS[name]
    d, H, hd = 4096, 32, 128
    gen = torch.Generator(device="cuda").manual_seed(7)
    w = {k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
         for k, s in dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(512, d), w_up=(512, d), w_down=(d, 512)).items()}
    kv = [[torch.randn((s, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)] for s, _ in step]
    xs = [torch.randn((n, d), device="cuda", generator=gen) for _, n in step]
    T, tol = sum(n for _, n in step), 2.0 ** -10 + 2.0 ** -9
    for target in (256, 255):
        m = HatMid(CFG, [w], n_pages=1600, io_dtype="f32", kv_dtype="f16", **LIMITS)
        m.kv_pool.fill_(0xFF)
        m.set_attn_targets(target, 2048)
        for dev, ((s, _), rows) in enumerate(zip(step, kv)):
            if s:
                m.kv_import(dev, 0, 0, *rows)
        m.forward([Segment(dev, hi.CHUNK, s, x) for dev, ((s, _), x) in enumerate(zip(step, xs))])
        q, o = (m.debug_dump(x, T).double().view(T, H, hd).transpose(0, 1).contiguous() for x in ("q", "attn"))
        t = 0
        for dev, (s, n) in enumerate(step):
            K, V = (x.double().transpose(0, 1).contiguous() for x in m.kv_export(dev, 0, 0, s + n))
            hidden = torch.arange(s + n, device="cuda")[None, :] > s + torch.arange(n, device="cuda")[:, None]
            b = torch.softmax((q[:, t:t + n] @ K.transpose(1, 2).contiguous() / hd ** 0.5).masked_fill(hidden, -float("inf")), -1) @ V
            a = o[:, t:t + n]
            err = (a - b).norm(dim=-1) / b.norm(dim=-1)
            assert bool(torch.isfinite(a).all()) and float((a - b).norm() / b.norm()) <= tol and float(err.max()) <= 4 * tol, (name, target, dev)
            t += n
        m.close()
