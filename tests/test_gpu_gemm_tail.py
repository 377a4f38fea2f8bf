"""GPU check of the O and down products whose last token tiles are split along K while the others stay whole."""
import ctypes as C

import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import to_np

pytestmark = pytest.mark.gpu
# 20 feature tiles of 256: from 13 token tiles of 256 rows on, one round of 256 workgroups leaves a remainder
CFG = dict(name="tail", n_layers=2, d_model=5120, n_heads=40, head_dim=128, d_ffn=13824, rms_eps=1e-6, rope_theta=1e4)
ROWS = [3213, 4037, 4096]      # ragged and whole last tiles, 8 and 3 pieces


def make(n_layers, T):
    import torch
    from paper_2503_18989_amd import HatMid
    gen = torch.Generator(device="cuda").manual_seed(T)
    d, f = CFG["d_model"], CFG["d_ffn"]
    shapes = dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(f, d), w_up=(f, d), w_down=(d, f))
    w = [{k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
          for k, s in shapes.items()} for _ in range(n_layers)]
    m = HatMid(dict(CFG, n_layers=n_layers), w, n_pages=8 * 40, max_devices=8, max_step_tokens=4096, max_pos=600, io_dtype="f32")
    n = [min(512, T - 512 * i) for i in range(8)]
    xs = [torch.randn((r, d), device="cuda", generator=gen) for r in n if r > 0]
    # the sizes are ones at which the planner splits the tail of both products
    for K in (d, f):
        tile, first, ks = (C.c_int32() for _ in range(3))
        assert m.lib.hat_mid_debug_gemm_split(T, 5120, d, K, 4096, C.byref(tile), C.byref(first), C.byref(ks)) == 0
        assert 0 < first.value < T and ks.value > 1, (T, K)
    return m, w, xs


@pytest.mark.parametrize("T", ROWS)
def test_split_tail_against_float64_products(T):
    # one layer: the dumps are the operands of O (attention output) and down (SwiGLU product), so that what the products
    # add, the norm between them and the last fold on the way out are known to fp32 sums: 13824 terms in fp32 chunks of the
    # matrix pipe are within 2^-24 * sqrt(13824) = 7e-6 of the sum's size (bounded here by 4e-5); the norm rounds to fp16
    import torch
    from paper_2503_18989_amd import Segment
    m, w, xs = make(1, T)
    outs = torch.cat(m.forward([Segment(i, hi.CHUNK, 0, x) for i, x in enumerate(xs)])).double()
    x = torch.cat(xs).double()
    attn, act, xn2 = (m.debug_dump(k, T).double() for k in ("attn", "act", "xnorm2"))
    mid = x + attn @ w[0]["wo"].double().T.contiguous()
    norm = mid * torch.rsqrt((mid ** 2).mean(1, keepdim=True) + CFG["rms_eps"]) * w[0]["ffn_norm"].double()
    assert float(((xn2 - norm).abs() / norm.abs().clamp_min(2.0 ** -6)).max()) <= 2.0 ** -10
    ref = mid + act @ w[0]["w_down"].double().T.contiguous()
    added = (ref - x).abs().max()
    assert float((outs - ref).abs().max() / added) <= 4e-5
    m.close()


@pytest.mark.parametrize("T", ROWS)
def test_split_tail_equals_unsplit_products(T):
    from paper_2503_18989_amd import Segment
    m, _, xs = make(CFG["n_layers"], T)

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
    # size; a lost or doubled partial sum moves it by an eighth or more.
    assert np.max(np.abs(planned - whole)) <= 2.0 ** -9 * np.max(np.abs(whole - x)) and np.all(np.isfinite(whole))
    m.close()
