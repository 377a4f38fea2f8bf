"""GPU check of the O and down products whose last token tiles are split along K while the others stay whole."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import to_np

pytestmark = pytest.mark.gpu
# 20 feature tiles of 256: from 13 token tiles on, one round of 256 workgroups leaves a remainder
CFG = dict(name="tail", n_layers=2, d_model=5120, n_heads=40, head_dim=128, d_ffn=2048, rms_eps=1e-6, rope_theta=1e4)


@pytest.mark.parametrize("T", [3400, 4000, 4096])      # ragged and whole last tiles
def test_split_tail_equals_unsplit_products(T):
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    gen = torch.Generator(device="cuda").manual_seed(T)
    d, f = CFG["d_model"], CFG["d_ffn"]
    shapes = dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(f, d), w_up=(f, d), w_down=(d, f))
    w = [{k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
          for k, s in shapes.items()} for _ in range(CFG["n_layers"])]
    m = HatMid(CFG, w, n_pages=8 * 40, max_devices=8, max_step_tokens=4096, max_pos=600, io_dtype="f32")
    n = [min(512, T - 512 * i) for i in range(8)]
    xs = [torch.randn((r, d), device="cuda", generator=gen) for r in n if r > 0]

    def step():
        outs = m.forward([Segment(i, hi.CHUNK, 0, x) for i, x in enumerate(xs)])
        return np.concatenate([to_np(o) for o in outs])
    planned, again = step(), step()
    assert np.array_equal(planned, again)
    for which in (1, 3):
        m.force_gemm(which, 19, 1)          # 256 x 256, every tile whole
    whole = step()
    x = np.concatenate([to_np(v) for v in xs])
    # fp32 sums in another order (2^-24 each) now and then flip the rounding of an operand element (fp16, 2^-11) and, in
    # the second layer, of a bf16 cache row (2^-9).  Every term of a sum off by a whole flip would move it by 2^-9 of its
    # size; a lost or doubled partial sum moves it by a third or more.
    assert np.max(np.abs(planned - whole)) <= 2.0 ** -9 * np.max(np.abs(whole - x)) and np.all(np.isfinite(whole))
    m.close()
