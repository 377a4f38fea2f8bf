"""GPU parity of chunk attention over few rows: items of at most 32 rows stream the cache where they are alone or one of them
is long, larger ones stage it."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import Pair, rel_err

pytestmark = pytest.mark.gpu
TOL = 6e-3          # at most 3 layers: the bar of test_gpu_parity.py
SHAPES = {64: dict(name="n64", n_layers=2, d_model=192, n_heads=3, head_dim=64, d_ffn=512, rms_eps=1e-6, rope_theta=1e4),
          128: dict(name="n128", n_layers=2, d_model=640, n_heads=5, head_dim=128, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)}


@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("target", [64, 4096])      # key ranges whole, and split as far as they go
def test_row_counts_around_the_edges(hd, kv, target):
    p = Pair(SHAPES[hd], 77, n_pages=8 * 100, max_devices=8, max_step_tokens=3200, max_pos=1600, kv_dtype=kv)
    p.gpu.set_attn_targets(target, target)
    rows = [1, 31, 32, 33, 16, 64, 65, 5]
    starts = [1540, 0, 15, 700, 31, 1023, 640, 900]

    def step(segs):
        for o, r in zip(*p.step(segs)):
            assert np.all(np.isfinite(o)) and rel_err(o, r) <= TOL, (segs, rel_err(o, r))
    step([(d, hi.CHUNK, 0, s) for d, s in enumerate(starts[:4]) if s])
    step([(d + 4, hi.CHUNK, 0, s) for d, s in enumerate(starts[4:]) if s])
    # narrow (the longest over 1541 keys) and wide chunks and a verify segment in one step; then a chunk whose last item is a narrow remainder
    step([(d, hi.CHUNK if d < 7 else hi.VERIFY, s, n) for d, (s, n) in enumerate(zip(starts, rows))])
    step([(1, hi.CHUNK, 20, 256 + 17), (3, hi.CHUNK, 690, 40)])
    step([(0, hi.CHUNK, 1541, 7), (2, hi.CHUNK, 47, 32), (4, hi.CHUNK, 40, 1)])      # narrow items only
    p.check_pages(range(8))
    p.close()


def test_split_key_ranges_lose_no_precision():
    # Against float64 attention over the same fp16 queries and bf16 cache rows, the fp16 rounding of the probabilities and of
    # the output are each about as large as the fp16 grid is coarse (u, relative to a row's output), whatever the split:
    # sqrt(2) u in all.  Partial results held in fp16 would add a third such term (sqrt(3) u, 1.22 times as much); held in
    # fp32 they add nothing that shows.  76 800 elements fix the ratio of the two rms errors to half a per cent.
    import torch
    from gpu_util import dev_weights
    from paper_2503_18989_amd import HatMid, Segment
    cfg = dict(SHAPES[128], n_layers=1)
    d, H, hd, n, starts = cfg["d_model"], cfg["n_heads"], cfg["head_dim"], 20, [1600, 1700, 1811, 1850, 1930, 2000]
    m = HatMid(cfg, [dev_weights(hi.layer_weights(cfg, 0, 3))], n_pages=6 * 130, max_devices=6, max_step_tokens=256, max_pos=2048, io_dtype="f32")
    gen = torch.Generator(device="cuda").manual_seed(5)
    for dev, s in enumerate(starts):
        k, v = (torch.randn((s, H, hd), device="cuda", generator=gen).bfloat16() for _ in range(2))
        m.kv_import(dev, 0, 0, k, v)
    xs = [torch.randn((n, d), device="cuda", generator=gen) for _ in starts]
    err = {}
    for target in (1, 2048):            # key ranges whole, and the library's own split (7 or 8 ranges)
        m.set_attn_targets(target, target)
        m.forward([Segment(dev, hi.CHUNK, s, x) for dev, (s, x) in enumerate(zip(starts, xs))])
        q = m.debug_dump("q", 6 * n).double().view(6, n, H, hd)
        o = m.debug_dump("attn", 6 * n).double().view(6, n, H, hd)
        total = 0.0
        for dev, s in enumerate(starts):
            K, V = (t.double() for t in m.kv_export(dev, 0, 0, s + n))
            sc = torch.stack([q[dev][:, h] @ K[:, h].T.contiguous() for h in range(H)], 1) / hd ** 0.5
            hidden = torch.arange(s + n, device="cuda")[None, None, :] > s + torch.arange(n, device="cuda")[:, None, None]
            p = torch.softmax(sc.masked_fill(hidden, -float("inf")), -1)
            ref = torch.stack([p[:, h] @ V[:, h].contiguous() for h in range(H)], 1)
            total += float(((o[dev] - ref) ** 2).sum() / (ref ** 2).sum())
        err[target] = (total / 6) ** 0.5
    assert err[2048] <= 1.08 * err[1] and err[1] <= 2.0 ** -11, err
    m.close()
