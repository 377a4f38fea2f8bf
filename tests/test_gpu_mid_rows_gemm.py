"""GPU check of the products of 257 .. 384 rows, whose token tiles may be 160, 192 or 224 rows tall (which of these steps have such
tiles: test_gemm_planner.py)."""
import pytest

from gpu_util import progress, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,heads", [(4096, 11008, 32), (2048, 5504, 32)])
@pytest.mark.parametrize("T", [257, 320, 321, 383, 384])      # both edges of the range, of two 160-row tiles, a last row of a 192-row one
def test_chosen_tiles_against_128_rows(d, f, heads, T):
    """One layer with the tiles that the planner chooses against the same layer in whole 128 x 128 tiles.  Only the order of fp32
    sums differs, which now and then moves an fp16 operand of the next product by its last place (2^-10 of it at most): what
    the layer adds to its input agrees to less than that in the 2-norm."""
    import torch
    from paper_2503_18989_amd import CHUNK, HatMid, Segment
    g = torch.Generator(device="cuda").manual_seed(T)
    def mat(n, k, std=0.02):
        return torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    one = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    w = dict(attn_norm=one, ffn_norm=one, wq=mat(d, d), wk=mat(d, d), wv=mat(d, d), wo=mat(d, d), w_gate=mat(f, d), w_up=mat(f, d), w_down=mat(d, f))
    m = HatMid(dict(n_layers=1, d_model=d, n_heads=heads, head_dim=d // heads, d_ffn=f, rms_eps=1e-6, rope_theta=1e4), [w], n_pages=32,
               max_devices=1, max_step_tokens=384, max_pos=512, io_dtype="f32")
    x = torch.empty((T, d), device="cuda").normal_(0, 1, generator=g)
    def added():
        return to_np(m.forward([Segment(0, CHUNK, 0, x)])[0] - x)
    got = added()
    for which in range(4):
        m.force_gemm(which, 4, 1)
    e = rel_l2(got, added())
    progress("tiles of %d rows, d = %d: %.2e against 128 x 128" % (T, d, e))
    assert e <= 2.0 ** -10
    m.close()
