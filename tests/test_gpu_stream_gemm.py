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
