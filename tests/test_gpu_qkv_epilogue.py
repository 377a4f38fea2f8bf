"""GPU check of the rotation and append in the QKV product's epilogue, for every LDS tile, against the rotary launch of its own."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import dev_weights, to_np

pytestmark = pytest.mark.gpu
APART = 1          # the forced tile whose QKV product leaves rotation and append to a launch
CFGS = [dict(name="hd64", n_layers=1, d_model=320, n_heads=5, head_dim=64, d_ffn=64, rms_eps=1e-6, rope_theta=1e4),      # 960 rows of W: every tile ragged
        dict(name="hd128", n_layers=1, d_model=384, n_heads=3, head_dim=128, d_ffn=64, rms_eps=1e-6, rope_theta=1e4)]


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("cfg", CFGS, ids=["hd64", "hd128"])
def test_every_lds_tile_rotates_and_appends(cfg, kv):
    """Segments that begin and end inside pages and cross the tiles' token blocks.  The rotary launch rounds q, k and v to fp16 on their
    way: 2^-12 of a value, which moves an element by at most one step of its type (the exported bf16: 2^-7 of its binade's lower end).
    Rows that are not new stay bit for bit."""
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    H, hd, starts, rows = cfg["n_heads"], cfg["head_dim"], [0, 3, 40, 17], [97, 160, 31, 225]
    w = dev_weights(hi.layer_weights(cfg, 0, 4))
    gen = torch.Generator(device="cuda").manual_seed(1)
    old = [torch.randn((64, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)]
    xs = [torch.from_numpy(hi.hidden_rows(n, cfg["d_model"], 4, 0, i)).cuda() for i, n in enumerate(rows)]
    m = HatMid(cfg, [w], n_pages=64, max_devices=4, max_step_tokens=sum(rows), max_pos=512, io_dtype="f32", kv_dtype=kv)
    for dev in range(4):
        m.kv_import(dev, 0, 0, *old)
    kept = m.kv_export(0, 0, 0, 64)           # (an fp16 cache rounds the smallest of the imported values)

    def step(tile):
        m.force_gemm(0, tile, 1)
        m.forward([Segment(i, hi.CHUNK, s, x) for i, (s, x) in enumerate(zip(starts, xs))])
        out = [to_np(m.debug_dump("q", sum(rows)))]
        for dev, (s, n) in enumerate(zip(starts, rows)):
            k, v = m.kv_export(dev, 0, 0, s + n)
            assert torch.equal(k[:s], kept[0][:s]) and torch.equal(v[:s], kept[1][:s]), tile
            out += [to_np(k[s:]), to_np(v[s:])]
        return out

    ref = step(APART)
    for tile in [-1] + [t for t in range(24) if t != APART]:
        for a, b in zip(step(tile), ref):
            assert np.max(np.abs(a - b)) <= 2.0 ** -7 * np.max(np.abs(b)), tile
    m.close()


def test_queries_of_a_step_beyond_two_to_the_31_elements():
    """91200 rows of the widest model: q, k and v of the rows from 87381 on lie more than 2^31 elements into their buffer.  The first and the last
    devices of the batch against the same prompts one at a time (the bound of a shallow model, on what the layer added)."""
    import torch
    from gpu_util import added_err
    from paper_2503_18989_amd import HatMid, Segment
    d, n, devices = 8192, 912, 100
    assert 3 * d * n * (devices - 1) > 2 ** 31
    cfg = dict(n_layers=1, d_model=d, n_heads=64, head_dim=128, d_ffn=64, rms_eps=1e-6, rope_theta=1e4)
    gen = torch.Generator(device="cuda").manual_seed(6)
    shapes = dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(64, d), w_up=(64, d), w_down=(d, 64))
    w = {k: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(float(len(s) == 1), 0.02, generator=gen) for k, s in shapes.items()}
    x = torch.empty((devices, n, d), device="cuda").normal_(generator=gen)
    m = HatMid(cfg, [w], n_pages=devices * 57, max_devices=devices, max_step_tokens=devices * n, max_pos=n, io_dtype="f32")
    got = m.forward([Segment(i, hi.CHUNK, 0, x[i]) for i in range(devices)])
    torch.cuda.synchronize()
    assert all(bool(torch.isfinite(y).all()) for y in got)
    one = HatMid(cfg, [w], n_pages=57, max_devices=1, max_step_tokens=n, max_pos=n, io_dtype="f32")
    for i in (0, 1, devices - 2, devices - 1):
        ref = one.forward([Segment(0, hi.CHUNK, 0, x[i])])[0]
        assert added_err(to_np(got[i]), to_np(ref), to_np(x[i])) <= 6e-3, i
    m.close()
    one.close()
