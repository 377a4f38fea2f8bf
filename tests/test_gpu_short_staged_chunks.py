"""Staged chunk items of few keys over an fp16 cache: which kernel takes them, and both kernels' attention against float64 softmax on either side of the line."""
import pytest

import hat_inputs as hi

CASES = {   # head dim: (rows of each device's chunk, keys before it), the last of the staged steps below the line and the first ones above it
    128: [(64, 0, False), (40, 50, False), (95, 0, False), (96, 0, True), (40, 56, True), (250, 100, True)],
    64: [(128, 0, False), (200, 55, False), (255, 0, False), (256, 0, True), (40, 216, True), (250, 300, True)],
}


def planned(hd, H, segs, target, kv="f16"):
    """(staged items taken by the ring kernel, workgroup waves of streamed ones)"""
    from paper_2503_18989_amd import HatPlanner
    cfg = dict(n_layers=1, d_model=H * hd, n_heads=H, head_dim=hd, d_ffn=256, rms_eps=1e-6, rope_theta=1e4)
    p = HatPlanner(cfg, 2000, max_devices=16, max_step_tokens=2560, max_pos=1024, kv_dtype=kv)
    p.set_attn_targets(target, 2048)
    if any(s for s, _ in segs):
        p.plan([(d, hi.CHUNK, 0, s) for d, (s, _) in enumerate(segs) if s])
    p.plan([(d, hi.CHUNK, s, n) for d, (s, n) in enumerate(segs)])
    r = p.staged_ring(), p.block_waves()
    p.close()
    return r


@pytest.mark.parametrize("hd", [64, 128])
def test_items_of_few_keys_do_not_take_the_ring(hd):
    for rows, start, ring in CASES[hd]:
        assert planned(hd, 8, [(start, rows)] * 4, 255) == (ring, 0), (rows, start)
        assert planned(hd, 8, [(start, rows)] * 4, 255, kv="bf16") == (False, 0)
    # eight new prompts of 128 rows at once stage by themselves: on average as many keys as they have rows
    assert planned(hd, 64, [(0, 128)] * 8, 256) == (hd == 128, 0)
    # an item of many keys makes up for one of few
    assert planned(hd, 8, [(0, 40), (900, 100)], 255)[0]


@pytest.mark.gpu
@pytest.mark.parametrize("hd", [64, 128])
def test_both_kernels_against_float64(hd):
    # probabilities, the partial results of key ranges and the output are rounded to fp16 once each, sqrt(3) * 2^-11.5 of a row's size in all, bounded by 2^-10.  The cached rows
    # are bf16 numbers; those of the step itself are exported rounded to bf16, 2^-9 of each of them, which is added where they are all there is
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    d, H = 512, 512 // hd
    cfg = dict(name="short", n_layers=1, d_model=d, n_heads=H, head_dim=hd, d_ffn=256, rms_eps=1e-6, rope_theta=1e4)
    gen = torch.Generator(device="cuda").manual_seed(hd)
    w = {k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
         for k, s in dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(256, d), w_up=(256, d), w_down=(d, 256)).items()}
    for rows, start, ring in CASES[hd]:
        assert planned(hd, H, [(start, rows)] * 4, 255) == (ring, 0)
        m = HatMid(cfg, [w], n_pages=200, max_devices=4, max_step_tokens=1024, max_pos=1024, io_dtype="f32", kv_dtype="f16")
        m.kv_pool.fill_(0xFF)          # NaN in every cache element that nothing has written
        m.set_attn_targets(255, 2048)
        if start:
            for dev in range(4):
                m.kv_import(dev, 0, 0, *(torch.randn((start, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)))
        m.forward([Segment(dev, hi.CHUNK, start, torch.randn((rows, d), device="cuda", generator=gen)) for dev in range(4)])
        q, o = (m.debug_dump(x, 4 * rows).double().view(4, rows, H, hd) for x in ("q", "attn"))
        hidden = torch.arange(start + rows, device="cuda")[None, :] > start + torch.arange(rows, device="cuda")[:, None]
        for dev in range(4):
            K, V = (x.double() for x in m.kv_export(dev, 0, 0, start + rows))
            for h in range(H):
                s = ((q[dev, :, h] @ K[:, h].T.contiguous()) / hd ** 0.5).masked_fill(hidden, -float("inf"))
                ref = torch.softmax(s, -1) @ V[:, h].contiguous()
                assert float((o[dev, :, h] - ref).norm() / ref.norm()) <= 2.0 ** -10 + 2.0 ** -9, (rows, start, dev, h)
        m.close()
