"""GPU check of the GEMM tiles whose weights and activations are brought by loader waves, at the edges of their rings: fewer k-tiles than a ring holds, one more
and one less than whole groups, ragged feature and token tiles, K split into pieces of a few k-tiles."""
import pytest

from gpu_util import progress, rel_l2, to_np

pytestmark = pytest.mark.gpu
LOADER_TILES = (2, 4, 5, 6, 7, 8, 9, 11, 12, 14, 15, 16, 18, 23)     # W loaded in groups of 2 .. 6 k-tiles
PLAIN = 13                                                           # 192 x 128, whose multiplying waves load


@pytest.mark.parametrize("d,f", [(64, 128), (192, 320), (320, 704), (576, 832), (832, 1600)])      # 1 .. 13 and 2 .. 25 k-tiles of 64
def test_loader_tiles_against_a_plain_one(d, f):
    """Only the order of fp32 sums differs, which now and then moves an fp16 operand of the next product by its last place: what
    the layer adds to its input agrees to 2^-10 in the 2-norm."""
    import torch
    from paper_2503_18989_amd import CHUNK, HatMid, Segment
    g = torch.Generator(device="cuda").manual_seed(d)
    def mat(n, k, std=0.05):
        return torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    one = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    w = dict(attn_norm=one, ffn_norm=one, wq=mat(d, d), wk=mat(d, d), wv=mat(d, d), wo=mat(d, d), w_gate=mat(f, d), w_up=mat(f, d), w_down=mat(d, f))
    m = HatMid(dict(n_layers=1, d_model=d, n_heads=d // 64, head_dim=64, d_ffn=f, rms_eps=1e-6, rope_theta=1e4), [w], n_pages=64,
               max_devices=1, max_step_tokens=768, max_pos=768, io_dtype="f32")
    for T in (1, 33, 160, 257, 513):
        x = torch.empty((T, d), device="cuda").normal_(0, 1, generator=g)
        def added(tile, ks):
            for which in range(4):
                m.force_gemm(which, tile, ks)
            return to_np(m.forward([Segment(0, CHUNK, 0, x)])[0] - x)
        ref = added(PLAIN, 1)
        worst = 0.0
        for tile in LOADER_TILES:
            for ks in (1, 3):
                e = rel_l2(added(tile, ks), ref)
                worst = max(worst, e)
                assert e <= 2.0 ** -10, (T, tile, ks, e)
        progress("loader tiles, d = %d, %d rows: %.2e" % (d, T, worst))
    m.close()
