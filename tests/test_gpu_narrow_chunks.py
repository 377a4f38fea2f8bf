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
    p = Pair(SHAPES[hd], 77, n_pages=8 * 90, max_devices=8, max_step_tokens=2600, max_pos=1400, kv_dtype=kv)
    p.gpu.set_attn_targets(target, target)
    rows = [1, 31, 32, 33, 16, 64, 65, 5]
    starts = [1030, 0, 15, 700, 31, 1023, 640, 900]

    def step(segs):
        for o, r in zip(*p.step(segs)):
            assert np.all(np.isfinite(o)) and rel_err(o, r) <= TOL, (segs, rel_err(o, r))
    step([(d, hi.CHUNK, 0, s) for d, s in enumerate(starts[:4]) if s])
    step([(d + 4, hi.CHUNK, 0, s) for d, s in enumerate(starts[4:]) if s])
    # narrow (the longest over 1031 keys) and wide chunks and a verify segment in one step; then a chunk whose last item is a narrow remainder
    step([(d, hi.CHUNK if d < 7 else hi.VERIFY, s, n) for d, (s, n) in enumerate(zip(starts, rows))])
    step([(1, hi.CHUNK, 20, 256 + 17), (3, hi.CHUNK, 690, 40)])
    step([(0, hi.CHUNK, 1031, 7), (2, hi.CHUNK, 47, 32), (4, hi.CHUNK, 40, 1)])      # narrow items only
    p.check_pages(range(8))
    p.close()
