"""Attention where the cache rows that nothing has written hold NaN, in every kernel: caches that end on each row of a page, in stages and key ranges of which
most pages are not the device's."""
import pytest

import hat_inputs as hi

CFG = {hd: dict(name="stale", n_layers=1, d_model=512, n_heads=512 // hd, head_dim=hd, d_ffn=256, rms_eps=1e-6, rope_theta=1e4) for hd in (64, 128)}
LIMITS = dict(max_devices=16, max_step_tokens=800, max_pos=1024)
WAYS = {"streamed": (hi.CHUNK, 45, 256), "staged": (hi.CHUNK, 45, 255), "narrow": (hi.CHUNK, 17, 256), "verify": (hi.VERIFY, 5, 256)}
START = 300       # + device


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("kv", ["bf16", "f16"])
def test_the_ways_are_those_meant(hd, kv):
    from paper_2503_18989_amd import HatPlanner
    for way, (kind, n, target) in WAYS.items():
        p = HatPlanner(CFG[hd], 400, kv_dtype=kv, **LIMITS)
        p.set_attn_targets(target, 2048)
        for dev in range(16):
            p.plan([(dev, hi.CHUNK, 0, START + dev)])
        r = p.plan([(dev, kind, START + dev, n) for dev in range(16)])
        assert (len(r["verify_items"]) > 0) == (way == "verify")
        assert p.narrow_items() == (len(r["chunk_items"]) if way == "narrow" else 0)
        assert (p.block_waves() in (4, 8)) == (way == "streamed")
        assert p.staged_ring() == (way == "staged" and kv == "f16")
        p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("way", list(WAYS))
@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
def test_rows_that_nothing_has_written_do_not_show(hd, kv, way):
    # probabilities, partial results and output rounded to fp16 once each, sqrt(3) * 2^-11.5 of a row's size; the step's own rows, a sixth of the keys, are exported rounded to
    # bf16 from an fp16 cache, 2^-9 of each: bounded by 2^-10 + 2^-9
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    kind, n, target = WAYS[way]
    cfg = CFG[hd]
    d, H = 512, cfg["n_heads"]
    gen = torch.Generator(device="cuda").manual_seed(hd)
    w = {k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
         for k, s in dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(256, d), w_up=(256, d), w_down=(d, 256)).items()}
    m = HatMid(cfg, [w], n_pages=400, io_dtype="f32", kv_dtype=kv, **LIMITS)
    m.kv_pool.fill_(0xFF)          # a NaN in every bf16 and fp16 element
    m.set_attn_targets(target, 2048)
    for dev in range(16):
        m.kv_import(dev, 0, 0, *(torch.randn((START + dev, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)))
    m.forward([Segment(dev, kind, START + dev, torch.randn((n, d), device="cuda", generator=gen)) for dev in range(16)])
    q, o = (m.debug_dump(x, 16 * n).double().view(16, n, H, hd).transpose(1, 2).contiguous() for x in ("q", "attn"))
    for dev in range(16):
        keys = START + dev + n
        K, V = (x.double().transpose(0, 1).contiguous() for x in m.kv_export(dev, 0, 0, keys))
        hidden = torch.arange(keys, device="cuda")[None, :] > START + dev + torch.arange(n, device="cuda")[:, None]
        ref = torch.softmax((q[dev] @ K.transpose(1, 2).contiguous() / hd ** 0.5).masked_fill(hidden, -float("inf")), -1) @ V
        assert bool(torch.isfinite(o[dev]).all()) and float((o[dev] - ref).norm() / ref.norm()) <= 2.0 ** -10 + 2.0 ** -9, dev
    m.close()
