"""GPU check that a row of a small batch is normalised in one stated order of fp32 operations, whichever launch does it."""
import numpy as np
import pytest

import hat_inputs as hi
from gpu_util import dev_weights, to_np

pytestmark = pytest.mark.gpu
F = np.float32


def norm_row_bits(x, gain, eps):
    """rmsnorm of fp32 rows, operation by operation: thread i of 256 holds octets i, i + 256, ..; each adds fma(a, a, b * b) for
    features e of the lower half (a) and upper half (b) of an octet; 64 lanes meet pairwise, then the four waves in order."""
    T, d = x.shape
    octs = np.zeros((T, 4 * 256, 2, 4), F)
    octs[:, :d // 8] = x.reshape(T, d // 8, 2, 4)
    octs = octs.reshape(T, 4, 256, 2, 4)
    ss = np.zeros((T, 256), F)
    for v in range(4):
        live = np.arange(256) + 256 * v < d // 8
        for e in range(4):
            a, b = octs[:, v, :, 0, e], octs[:, v, :, 1, e]
            term = (np.longdouble(a) * np.longdouble(a) + np.longdouble(b * b)).astype(F)   # (a^2 is exact in 64 bits)
            ss = np.where(live, ss + term, ss)
    w = ss.reshape(T, 4, 64)
    for o in (32, 16, 8, 4, 2, 1):
        w = w[:, :, :o] + w[:, :, o:2 * o]
    w = w[:, :, 0]
    total = ((w[:, 0] + w[:, 1]) + w[:, 2]) + w[:, 3]
    r = F(1) / np.sqrt(total / F(d) + F(eps))
    return np.clip(x * r[:, None] * gain[None, :], F(-65504), F(65504)).astype(np.float16)


@pytest.mark.parametrize("profiled", [False, True])       # the first norm in the gather launch, and as a launch of its own
@pytest.mark.parametrize("d,heads,T", [(192, 3, 5), (2048, 32, 1023), (4096, 32, 900), (5120, 40, 600), (8192, 64, 97)])
def test_first_norm_bits(d, heads, T, profiled):
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    cfg = dict(name="n", n_layers=1, d_model=d, n_heads=heads, head_dim=d // heads, d_ffn=64, rms_eps=1e-6, rope_theta=1e4)
    w = hi.layer_weights(cfg, 0, 5, gain_jitter=0.1)
    m = HatMid(cfg, [dev_weights(w)], n_pages=64, max_devices=1, max_step_tokens=1024, max_pos=1024, io_dtype="f32")
    x = np.random.default_rng(T).standard_normal((T, d), dtype=F)      # (squares of bf16 values would be exact in any order)
    m.set_profiling(profiled)
    m.forward([Segment(0, hi.CHUNK, 0, torch.from_numpy(x).cuda())])
    got = to_np(m.debug_dump("xnorm", T)).astype(np.float16)
    gain = to_np(dev_weights(w)["attn_norm"]).astype(F)
    assert np.array_equal(got, norm_row_bits(x, gain, cfg["rms_eps"]))
    m.close()


@pytest.mark.parametrize("d,T", [(192, 5), (2112, 33), (4160, 5), (6208, 17), (8192, 3),    # one to four octets per thread, ragged and whole
                                 (1024, 33),                                                # one octet, enough of K for the second group of four
                                 (4160, 513), (6208, 513)])                                 # wide rows beyond 512: one sum at a time
def test_norm_folds_partial_sums(d, T):
    """The second norm adds the O product's partial sums (none, one group of four loads, a group and a remainder) to the residual.  A
    zero down projection hands that residual out, so its norm can be stated bit for bit.  Against the unsplit product only the order
    of the fp32 sums over K changes: each of the K terms' additions rounds by at most 2^-24 of the sum of their sizes."""
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    heads, f = d // 64, 64
    cfg = dict(name="n", n_layers=1, d_model=d, n_heads=heads, head_dim=64, d_ffn=f, rms_eps=1e-6, rope_theta=1e4)
    g = torch.Generator().manual_seed(d)
    def mat(n, k):
        return torch.randn((n, k), generator=g).mul_(0.02).to(torch.bfloat16)
    w = dict(attn_norm=torch.ones(d, dtype=torch.bfloat16), ffn_norm=(1 + 0.1 * torch.randn(d, generator=g)).to(torch.bfloat16), wq=mat(d, d),
             wk=mat(d, d), wv=mat(d, d), wo=mat(d, d), w_gate=mat(f, d), w_up=mat(f, d), w_down=torch.zeros((d, f), dtype=torch.bfloat16))
    m = HatMid(cfg, [{k: v.cuda() for k, v in w.items()}], n_pages=8 + T // 16, max_devices=1, max_step_tokens=64 + T, max_pos=128 + T, io_dtype="f32")
    x = torch.randn((T, d), generator=g)
    whole = bound = None
    for ks in (1, 2, 3, 4, 5, 6):
        m.force_gemm(1, 4, ks)
        out = to_np(m.forward([Segment(0, hi.CHUNK, 0, x.cuda())])[0]).astype(F)
        got = to_np(m.debug_dump("xnorm2", T)).astype(np.float16)
        assert np.array_equal(got, norm_row_bits(out, w["ffn_norm"].float().numpy(), cfg["rms_eps"])), ks
        if whole is None:
            attn = np.abs(to_np(m.debug_dump("attn", T)).astype(np.float64))
            whole, bound = out, 2.0 ** -24 * d * (attn @ np.abs(w["wo"].float().numpy().astype(np.float64)).T + np.abs(x.numpy()))
        assert np.all(np.abs(out.astype(np.float64) - whole) <= 2 * bound), ks
    m.close()
