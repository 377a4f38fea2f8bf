"""GPU parity of the weight-streaming GEMM at the edges of its tiles and of its K split among the waves."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import Pair, added_err, rel_err, to_np

pytestmark = pytest.mark.gpu
TOL = 6e-3          # one layer, fp32 I/O: the bar of test_gpu_parity.py, also against what the layer added
STREAM_TILES = (24, 25, 26, 27)
# K = 320 / 704: 20 and 44 k-steps for up to 32 wave shares (some of them empty); K = 4096: shares longer than the ring
CFGS = [dict(name="k320", n_layers=1, d_model=320, n_heads=5, head_dim=64, d_ffn=700, rms_eps=1e-6, rope_theta=1e4),
        dict(name="k4096", n_layers=1, d_model=4096, n_heads=32, head_dim=128, d_ffn=1000, rms_eps=1e-6, rope_theta=1e4)]


@pytest.mark.parametrize("cfg", CFGS, ids=["k320", "k4096"])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 64, 65, 96, 97])
def test_streaming_tiles_forced_and_planned(cfg, T):
    import torch
    from paper_2503_18989_amd import Segment
    p = Pair(cfg, 31 + T, n_pages=16, io_dtype="f32", max_devices=1, max_step_tokens=128, max_pos=128)
    x = hi.hidden_rows(T, cfg["d_model"], 31, T, 0)
    ref = p.ref.forward([(0, 0, x)])[0]
    xd = torch.from_numpy(x).cuda()
    for tile, ks in [(-1, 0)] + [(t, k) for t in STREAM_TILES for k in (1, 3, 4)]:
        for which in range(4):
            p.gpu.force_gemm(which, tile, ks)
        out = to_np(p.gpu.forward([Segment(0, hi.CHUNK, 0, xd)])[0])
        assert np.all(np.isfinite(out)), (tile, ks)
        e, ea = rel_err(out, ref), added_err(out, ref, x)
        assert e <= TOL and ea <= TOL, "tile %d ksplit %d: %.3e, vs added %.3e" % (tile, ks, e, ea)
    p.close()


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("cfg", CFGS, ids=["k320", "k4096"])
def test_rows_beyond_the_fp16_range_saturate_as_in_larger_batches(cfg, kv):
    # q, k and v beyond +-65504 are clamped there before anything else happens to them, whether the product that makes them
    # also rotates and appends (up to 96 rows) or not (97 rows).  Both round what they clamp: to fp16 once more in the
    # larger batch (2^-11 of 65504 an element, sqrt(2) times that after the rotation), to the cache type (2^-9 for bf16).
    import torch
    from gpu_util import dev_weights
    from paper_2503_18989_amd import HatMid, Segment
    w = hi.layer_weights(cfg, 0, 9)
    w = {k: v * np.float32(2.0 ** 20) if k in ("wq", "wk", "wv") else v for k, v in w.items()}
    x = torch.from_numpy(hi.hidden_rows(97, cfg["d_model"], 9, 0, 0)).cuda()
    rows = {}
    for T in (97, 1, 32, 64, 96):
        m = HatMid(cfg, [dev_weights(w)], n_pages=8, max_devices=1, max_step_tokens=128, max_pos=128, io_dtype="f32", kv_dtype=kv)
        m.forward([Segment(0, hi.CHUNK, 0, x[:T])])
        rows[T] = [to_np(m.debug_dump("q", T))] + [to_np(t).reshape(T, -1) for t in m.kv_export(0, 0, 0, T)]
        m.close()
        assert np.max(np.abs(rows[97][2])) == 65536, "the inputs were meant to exceed the range (65504 is 65536 in bf16)"
        for name, got, ref in zip("qkv", rows[T], rows[97]):
            assert np.max(np.abs(got - ref[:T])) <= 2.0 ** -7 * 65536, (name, T)


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("cfg", CFGS, ids=["hd64", "hd128"])
@pytest.mark.parametrize("tile", STREAM_TILES)
def test_rotation_and_append_inside_the_product_equal_the_separate_launch(cfg, kv, tile):
    # every streaming tile, over ragged segments that begin and end inside pages and cross token tiles: queries and cache
    # rows against those of an LDS tile with its own rotary launch (to one rounding: the fp16 one on the way, 2^-12 of a value,
    # moves an element by at most one step of its type, the exported bf16 by 2^-7 of its binade's lower end); rows of the
    # pages that are not new stay bit for bit
    import torch
    from gpu_util import dev_weights
    from paper_2503_18989_amd import HatMid, Segment
    H, hd, starts, rows = cfg["n_heads"], cfg["head_dim"], [0, 3, 40, 17], [1, 30, 14, 53]
    w = dev_weights(hi.layer_weights(cfg, 0, 4))
    gen = torch.Generator(device="cuda").manual_seed(tile)
    old = [torch.randn((96, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2)]
    xs = [torch.from_numpy(hi.hidden_rows(n, cfg["d_model"], 4, 0, i)).cuda() for i, n in enumerate(rows)]
    got = {}
    for forced in (1, tile):
        m = HatMid(cfg, [w], n_pages=40, max_devices=4, max_step_tokens=128, max_pos=128, io_dtype="f32", kv_dtype=kv)
        for dev in range(4):
            m.kv_import(dev, 0, 0, *old)
        kept = m.kv_export(0, 0, 0, 96)       # (an fp16 cache rounds the smallest of the imported values)
        m.force_gemm(0, forced, 1)
        m.set_profiling(True)
        m.forward([Segment(i, hi.CHUNK, s, x) for i, (s, x) in enumerate(zip(starts, xs))])
        torch.cuda.synchronize()
        assert m.kernel_times()["rope_append"][1] == (2 if forced == 1 else 1)     # the rotary table, and the launch per layer
        got[forced] = [to_np(m.debug_dump("q", sum(rows)))]
        for dev, (s, n) in enumerate(zip(starts, rows)):
            k, v = m.kv_export(dev, 0, 0, s + n)
            assert torch.equal(k[:s], kept[0][:s]) and torch.equal(v[:s], kept[1][:s])
            got[forced] += [to_np(k[s:]), to_np(v[s:])]
        m.close()
    for a, b in zip(got[tile], got[1]):
        assert np.max(np.abs(a - b)) <= 2.0 ** -7 * np.max(np.abs(b))
