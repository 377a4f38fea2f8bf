"""Attention against float64 softmax where the reference that a row's sums are kept against has to move: score sizes that grow or
shrink along the keys, by less than the slack (2^8) a tile and by more, staged, streamed in row blocks and as verify rows."""
import pytest

import hat_inputs as hi

pytestmark = pytest.mark.gpu


# Probabilities, the partial results of key ranges and the output are rounded to fp16 once each: sqrt(3) * 2^-11.5 of a row's size in all, bounded
# by 2^-10.  The cached keys and values are bf16 numbers in either cache type.  A step's own rows an fp16 cache exports rounded
# to bf16: their scores lie some 20 (log2) below the largest ones of the cached keys, so that does not show.
@pytest.mark.parametrize("kv", ["bf16", "f16"])
@pytest.mark.parametrize("hd", [64, 128])
def test_scores_that_grow_or_shrink_along_the_keys(hd, kv):
    import torch
    from paper_2503_18989_amd import HatMid, Segment
    d, start = 2048, 1207
    H = d // hd
    cfg = dict(name="slack", n_layers=1, d_model=d, n_heads=H, head_dim=hd, d_ffn=512, rms_eps=1e-6, rope_theta=1e4)
    gen = torch.Generator(device="cuda").manual_seed(hd)
    w = {k: torch.randn(s, device="cuda", generator=gen).mul_(0.02).add_(1.0 if k.endswith("norm") else 0.0).bfloat16()
         for k, s in dict(attn_norm=(d,), wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), ffn_norm=(d,), w_gate=(512, d), w_up=(512, d), w_down=(d, 512)).items()}
    pos = torch.arange(start, device="cuda", dtype=torch.float32)
    sizes = dict(up=0.05 * 300.0 ** (pos / start), down=15.0 * 300.0 ** (-pos / start), jumps=torch.where(pos.int() // 100 % 3 == 2, 12.0, 0.3))
    for name, size in sizes.items():
        for kind, rows, target in ((hi.CHUNK, 290, 256), (hi.CHUNK, 290, 64), (hi.CHUNK, 290, 4096), (hi.VERIFY, 7, 256)):
            m = HatMid(cfg, [w], n_pages=110, max_devices=1, max_step_tokens=320, max_pos=1600, io_dtype="f32", kv_dtype=kv)
            m.set_attn_targets(target, 2048)
            k, v = (torch.randn((start, H, hd), device="cuda", generator=gen) for _ in range(2))
            m.kv_import(0, 0, 0, (k * size[:, None, None]).bfloat16(), v.bfloat16())
            m.forward([Segment(0, kind, start, torch.randn((rows, d), device="cuda", generator=gen))])
            q, o = (m.debug_dump(x, rows).double().view(rows, H, hd) for x in ("q", "attn"))
            K, V = (x.double() for x in m.kv_export(0, 0, 0, start + rows))
            hidden = torch.arange(start + rows, device="cuda")[None, :] > start + torch.arange(rows, device="cuda")[:, None]
            for h in range(H):
                s = ((q[:, h] @ K[:, h].T.contiguous()) / hd ** 0.5).masked_fill(hidden, -float("inf"))
                ref = torch.softmax(s, -1) @ V[:, h].contiguous()
                assert float((o[:, h] - ref).norm() / ref.norm()) <= 2.0 ** -10, (name, kind, target, h)
            m.close()
