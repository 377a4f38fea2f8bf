"""GPU check of the rotation and append in the QKV product's epilogue, for every tile, to the bit: each weight row has one element, so that the
product is exact, and what is left is the rotation in fp32 and one rounding, which numpy repeats."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import dev_weights, to_np

pytestmark = pytest.mark.gpu
APART = 1          # the forced tile whose QKV product leaves rotation and append to a launch
TILES = 28
# 960 and 1152 rows of W, padded to 1024 and 1280: the last feature tile is partly or wholly padding in all but the heights that divide both
CFGS = [dict(name="hd64", n_layers=1, d_model=320, n_heads=5, head_dim=64, d_ffn=64, rms_eps=1e-6, rope_theta=1e4),
        dict(name="hd128", n_layers=1, d_model=384, n_heads=3, head_dim=128, d_ffn=64, rms_eps=1e-6, rope_theta=1e4)]


def one_element_rows(d, rng):
    """W with a single element +-1, +-0.5 or +-0.25 in each row, and x -> x W^T (exact in fp32)."""
    col, scale = rng.integers(0, d, d), rng.choice([1.0, -1.0, 0.5, -0.5, 0.25, -0.25], d).astype(np.float32)
    w = np.zeros((d, d), np.float32)
    w[np.arange(d), col] = scale
    return w, lambda x: x[:, col] * scale


def rotated(x, pos, cfg):
    """The rotation in fp32, the second product of each element rounded before the first is added to it (np.float64 holds a product and, but for
    sums 2^29 apart, the sum)."""
    H, hd = cfg["n_heads"], cfg["head_dim"]
    ang = pos[:, None].astype(np.float64) * np.float64(cfg["rope_theta"]) ** (-2.0 * np.arange(hd // 2) / hd)
    c, s = (f(ang).astype(np.float32)[:, None] for f in (np.cos, np.sin))
    a, b = np.split(x.reshape(-1, H, hd), 2, axis=2)
    fma = lambda p, q, r: (p.astype(np.float64) * q + r).astype(np.float32)
    return np.concatenate([fma(a, c, -(b * s)), fma(b, c, a * s)], axis=2)


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("cfg", CFGS, ids=["hd64", "hd128"])
def test_every_tile_rotates_and_appends(cfg, kv):
    """Segments that begin and end inside pages and cross the tiles' token blocks.  Rows that are not new stay bit for bit.  The rotary launch of
    its own may round the other product of an element first: one step of its type."""
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    H, hd, d, starts, rows = cfg["n_heads"], cfg["head_dim"], cfg["d_model"], [0, 3, 40, 17], [97, 160, 31, 225]
    rng = np.random.default_rng(5)
    w = hi.layer_weights(cfg, 0, 4)
    product = {}
    for name in ("wq", "wk", "wv"):
        w[name], product[name] = one_element_rows(d, rng)
    w = dev_weights(w)
    gen = torch.Generator(device="cuda").manual_seed(1)
    old = [torch.randn((64, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)]
    xs = [torch.from_numpy(hi.hidden_rows(n, d, 4, 0, i)).cuda() for i, n in enumerate(rows)]
    m = HatMid(cfg, [w], n_pages=64, max_devices=4, max_step_tokens=sum(rows), max_pos=512, io_dtype="f32", kv_dtype=kv)
    for dev in range(4):
        m.kv_import(dev, 0, 0, *old)
    kept = m.kv_export(0, 0, 0, 64)           # (an fp16 cache rounds the smallest of the imported values)

    def step(tile):
        m.force_gemm(0, tile, 1)
        m.forward([Segment(i, hi.CHUNK, s, x) for i, (s, x) in enumerate(zip(starts, xs))])
        q, new = to_np(m.debug_dump("q", sum(rows))), []
        for dev, (s, n) in enumerate(zip(starts, rows)):
            k, v = m.kv_export(dev, 0, 0, s + n)
            assert torch.equal(k[:s], kept[0][:s]) and torch.equal(v[:s], kept[1][:s]), tile
            new.append((k[s:], v[s:]))
        return [q] + [to_np(torch.cat(t)) for t in zip(*new)]

    got = {tile: step(tile) for tile in range(-1, TILES)}
    x = to_np(m.debug_dump("xnorm", sum(rows)))
    pos = np.concatenate([s + np.arange(n) for s, n in zip(starts, rows)])
    cached = lambda t: to_np(torch.from_numpy(t.astype(np.float16).astype(np.float32) if kv == "f16" else t).bfloat16())
    q, k = (rotated(product[name](x), pos, cfg) for name in ("wq", "wk"))
    want = [q.reshape(-1, d).astype(np.float16).astype(np.float32), cached(k), cached(product["wv"](x).reshape(-1, H, hd))]
    for tile in got:
        for a, b, ulp in zip(got[tile], want, (2.0 ** -10, 2.0 ** -7, 2.0 ** -7)):
            bad = np.abs(a - b) > ulp * np.abs(b) if tile == APART else a != b
            assert not bad.any(), (tile, ulp, int(bad.sum()), a[bad][:4], b[bad][:4])
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
