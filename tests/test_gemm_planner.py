"""Host logic of the GEMM launch planner (no GPU): its choices respect the contract of the kernels
for every shape of the workloads."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def lib():
    import os
    from paper_2503_18989_amd.binding import lib_path, load_library
    if not os.path.exists(lib_path()):
        from paper_2503_18989_amd.build import build
        build(verbose=False)
    return load_library()


def plan(lib, T, Nw, Nout, K, epi, part_rows):
    t, k = C.c_int32(-7), C.c_int32(-7)
    assert lib.hat_mid_debug_gemm_plan(T, Nw, Nout, K, epi, part_rows, C.byref(t), C.byref(k)) == 0
    return t.value, k.value


SHAPES = {   # name: (Nw, Nout, K, epilogue)   7B- and 13B-shaped layers, tiny
    "qkv7": (12288, 12288, 4096, 0), "o7": (4096, 4096, 4096, 2), "gu7": (22016, 11008, 4096, 1), "down7": (4096, 4096, 11008, 2),
    "qkv13": (15360, 15360, 5120, 0), "o13": (5120, 5120, 5120, 2), "gu13": (27648, 13824, 5120, 1), "down13": (5120, 5120, 13824, 2),
    "qkvT": (768, 768, 256, 0), "oT": (256, 256, 256, 2), "guT": (1536, 704, 256, 1), "downT": (256, 256, 704, 2),
}


@pytest.mark.parametrize("T", [1, 5, 32, 150, 256, 700, 1380, 3556, 5220, 8192])
def test_choices_are_launchable(lib, T):
    n_tiles = lib.hat_mid_debug_gemm_tile_count()
    for name, (Nw, Nout, K, epi) in SHAPES.items():
        for part_rows in (0, 4096):
            tile, ks = plan(lib, T, Nw, Nout, K, epi, part_rows)
            assert 0 <= tile < n_tiles, name
            assert ks >= 1
            if epi != 2 or part_rows == 0:
                assert ks == 1, "only the accumulating epilogue with a partial-sum buffer may split K (%s)" % name
            else:
                assert ks * T <= part_rows or ks == 1
                assert K // 64 // ks >= 1


def test_small_batches_split_k_and_large_ones_do_not(lib):
    # few token rows: the 4096 x 4096 projection has 16-32 feature tiles, so K is split to fill the CUs;
    # thousands of rows give enough tiles by themselves
    assert plan(lib, 256, 4096, 4096, 4096, 2, 4096)[1] > 1
    assert plan(lib, 3556, 4096, 4096, 4096, 2, 4096)[1] == 1
    assert plan(lib, 256, 4096, 4096, 4096, 2, 0)[1] == 1


def test_null_outputs_are_refused(lib):
    assert lib.hat_mid_debug_gemm_plan(256, 4096, 4096, 4096, 2, 4096, None, None) == -1


def tile_info(lib, tile):
    v = [C.c_int32(-1) for _ in range(5)]
    rc = lib.hat_mid_debug_gemm_tile_info(tile, *[C.byref(x) for x in v])
    return rc, tuple(x.value for x in v)


def test_tile_table_fits_the_hardware(lib):
    n = lib.hat_mid_debug_gemm_tile_count()
    assert n >= 20
    for t in range(n):
        rc, (bf, bt, waves, bk, ns) = tile_info(lib, t)
        assert rc == 0
        assert bf % 32 == 0 and bt % 32 == 0 and bk % 16 == 0 and 2 <= ns <= 4
        assert waves in (2, 4, 8)
        loaders, lds = C.c_int32(-1), C.c_int32(-1)
        assert lib.hat_mid_debug_gemm_tile_resources(t, C.byref(loaders), C.byref(lds)) == 0
        streaming = t >= n - 4
        if loaders.value:   # a ring of W that is longer than that of X
            assert not streaming and loaders.value == bk // 16 and lds.value > ns * (bf + bt) * bk * 2
        elif not streaming:
            assert lds.value == ns * (bf + bt) * bk * 2
        assert 0 < lds.value <= 160 * 1024, "rings of tile %d exceed the LDS of a CU" % t
        # accumulators (fp32, 64 lanes per wave) + operands must fit the register file of the waves' SIMDs, which the loader waves share
        acc_regs = bf * bt // (waves * 64)
        simd_waves = -(-(waves + loaders.value) // 4)
        assert acc_regs <= 512 // simd_waves - 56, "tile %d: %d accumulator registers per lane" % (t, acc_regs)
    assert lib.hat_mid_debug_gemm_tile_resources(n, None, None) == -1 and lib.hat_mid_debug_gemm_tile_resources(0, None, None) == 0
    assert tile_info(lib, n)[0] == -1 and tile_info(lib, -1)[0] == -1
    assert lib.hat_mid_debug_gemm_tile_info(0, None, None, None, None, None) == 0


def test_small_batches_keep_power_of_two_token_tiles_and_large_ones_use_the_big_tile(lib):
    for T in (1, 32, 128, 150, 161, 256):
        for name, (Nw, Nout, K, epi) in SHAPES.items():
            tile, _ = plan(lib, T, Nw, Nout, K, epi, 4096)
            bt = tile_info(lib, tile)[1][1]
            # the one exception: 129 .. 160 rows may take the 160-row token tile (one token tile instead of two)
            assert bt & (bt - 1) == 0 or (bt == 160 and 128 < T <= 160), "%s at T=%d took a %d-row token tile" % (name, T, bt)
    for name in ("gu7", "down7", "o13", "gu13", "down13"):     # 30 devices x 5 draft rows: the verify-heavy batch (O of the 7B shape measured faster with 64 x 256)
        Nw, Nout, K, epi = SHAPES[name]
        tile, _ = plan(lib, 150, Nw, Nout, K, epi, 4096)
        assert tile_info(lib, tile)[1][:2] == (128, 160), name
    for name in ("qkv7", "gu7", "qkv13", "gu13"):
        Nw, Nout, K, epi = SHAPES[name]
        tile, ks = plan(lib, 8192, Nw, Nout, K, epi, 4096)
        bf, bt, waves = tile_info(lib, tile)[1][:3]
        assert (bf, bt, waves, ks) == (256, 256, 8, 1), name
    # 2200 rows: 8.6 tiles of 256 rows; the 160-row tile (13.75 -> 14 tiles, 2 % padding instead of 5 %, and a tile count
    # that packs the 256 CUs better) measured 21-23 % faster on the O and down projections
    for name in ("o7", "down7"):
        Nw, Nout, K, epi = SHAPES[name]
        tile, ks = plan(lib, 2200, Nw, Nout, K, epi, 4096)
        assert tile_info(lib, tile)[1][1] in (160, 192)


WIDTHS = {   # d_model, d_ffn (padded to 64): the workloads' shapes, head-dim-64 shapes of middling width, the widest model accepted
    "tiny": (256, 704), "1k": (1024, 2816), "2k": (2048, 5504), "3k": (3072, 8192), "7b": (4096, 11008), "13b": (5120, 13824), "6k": (6144, 16384), "8k": (8192, 28672),
}


@pytest.mark.parametrize("name", list(WIDTHS))
def test_partial_sums_fit_their_buffer_at_every_batch_size(lib, name):
    d, f = WIDTHS[name]
    pad = lambda n: (n + 255) // 256 * 256
    for K in (d, f):
        for part_rows in (0, 100, 4096):
            for T in list(range(1, 400)) + list(range(400, 8193, 7)) + [512, 1024, 2048, 4096, 8192]:
                v = [C.c_int32(-7) for _ in range(3)]
                assert lib.hat_mid_debug_gemm_split(T, pad(d), d, K, part_rows, *[C.byref(x) for x in v]) == 0
                tile, first, ks = (x.value for x in v)
                bt = tile_info(lib, tile)[1][1]
                assert ks >= 1 and K // 64 // ks >= 1
                assert 0 <= first < T and first % bt == 0 and (first == 0 or ks > 1)
                assert ks == 1 or ks * (T - first) <= part_rows, (T, K, tile, first, ks)
                assert (tile, 1 if first else ks) == plan(lib, T, pad(d), d, K, 2, part_rows)
    assert lib.hat_mid_debug_gemm_split(256, 4096, 4096, 4096, 4096, None, None, None) == -1


@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 64, 65, 96, 97, 256])
def test_qkv_of_few_rows_takes_a_streaming_tile_built_for_it(lib, T):
    for name in ("qkv7", "qkv13", "qkvT"):
        Nw, Nout, K, _ = SHAPES[name]
        tile, ks = plan(lib, T, Nw, Nout, K, 3, 4096)
        assert ks == 1 and (24 <= tile < 28 if tile >= 0 else T > 16), (name, tile)
        if tile >= 0:
            bf, bt = tile_info(lib, tile)[1][:2]
            assert bt >= min(T, 32) and Nout % bf == 0
        plain, _ = plan(lib, T, Nw, Nout, K, 0, 4096)
        assert plain < 24                             # the plain product has LDS tiles only
    assert plan(lib, T, 12288, 12288, 4096, 3, 4096)[0] == (24 if T <= 16 else 27 if T <= 32 else 25 if T <= 64 else 26 if T <= 96 else -1)


def test_the_tail_is_split_only_where_it_is_predicted_to_win_clearly(lib):
    # measured in whole layers: at most 8 pieces, and not where the cost model's error exceeds its advantage
    def split(T, d, K):
        v = [C.c_int32() for _ in range(3)]
        assert lib.hat_mid_debug_gemm_split(T, d, d, K, 4096, *[C.byref(x) for x in v]) == 0
        return v[1].value, v[2].value
    for name, (d, f) in WIDTHS.items():
        for K in (d, f):
            for T in range(385, 4097):
                first, ks = split(T, d, K)
                assert first == 0 or ks <= 8, (name, K, T)
                assert first == 0 or name in ("13b", "6k", "8k"), (name, K, T)
    for T in (3213, 4037, 4096):
        assert split(T, 5120, 5120)[0] == 3072 and split(T, 5120, 13824)[0] == 3072


def test_qkv_tiles_of_wide_models_do_not_run_over_into_a_second_round(lib):
    for d, T, want in [(5120, 17, 27), (5120, 32, 27), (5504, 16, 24), (5504, 17, 24), (6144, 24, 24), (6144, 25, -1), (8192, 32, -1)]:
        N = (3 * d + 255) // 256 * 256
        assert plan(lib, T, N, 3 * d, d, 3, 4096)[0] == want, (d, T)


@pytest.mark.parametrize("T", [1, 16, 17, 24, 32, 33])
def test_o_and_down_of_a_narrow_model_stream_up_to_32_rows(lib, T):
    # 1024 x 2816: 32 panels in four pieces of K.  The 160 panels of the 13B shape stay whole and stream up to 16 rows
    for K in (1024, 2816):
        assert (plan(lib, T, 1024, 1024, K, 2, 4096) == (24, 4)) == (T <= 32)
    for K in (5120, 13824):
        assert (plan(lib, T, 5120, 5120, K, 2, 4096)[0] == 24) == (T <= 16)


def test_token_tiles_between_the_powers_of_two_from_257_rows_on(lib):
    # the steps of test_gpu_mid_rows_gemm.py: where a third 128-row token tile would be nearly empty, no product keeps it; 384 rows are two whole
    # 192-row tiles too, which gate/up of the wide models goes by (steps of the 13B shape 318 -> 304 us a layer), while 2048-wide models stay with 64, 128 and 256 rows there
    def token_rows(d, f, T):
        pad = lambda n: (n + 255) // 256 * 256
        return [tile_info(lib, plan(lib, T, pad(n), o, k, e, 4096)[0])[1][1]
                for n, o, k, e in ((3 * d, 3 * d, d, 0), (d, d, d, 2), (2 * f, f, d, 1), (d, d, f, 2))]
    for T in (257, 320):
        assert token_rows(4096, 11008, T) == [160] * 4
        assert 160 in token_rows(2048, 5504, T)
    assert 192 in token_rows(4096, 11008, 383) + token_rows(5120, 13824, 383)
    for d, f in ((4096, 11008), (5120, 13824), (8192, 28672)):
        assert token_rows(d, f, 384)[2] == 192, d
    assert all(bt in (64, 128, 256) for bt in token_rows(2048, 5504, 384))


@pytest.mark.parametrize("d,f,T,first,ks", [(5120, 13824, 3300, 3072, 8), (6144, 16384, 2788, 2560, 8), (8192, 28672, 2300, 2048, 8), (8192, 28672, 3300, 2048, 3)])
def test_tails_that_measured_faster_are_split(lib, d, f, T, first, ks):
    # down of these steps 4 .. 16 % faster than whole
    v = [C.c_int32() for _ in range(3)]
    assert lib.hat_mid_debug_gemm_split(T, d, d, f, 4096, *[C.byref(x) for x in v]) == 0
    assert tuple(x.value for x in v) == (19, first, ks)


def test_narrow_models_take_a_tile_without_loader_waves_from_257_rows_on(lib):
    # 128 x 64 rows, the multiplying waves load (tile 10): steps of 385 .. 1100 rows of these models measured 4 .. 7 % faster with it than with the tiles of loader waves.  Up to 256 rows it is not offered
    for name, (d, f) in WIDTHS.items():
        for N, o, K, e in ((3 * d, 3 * d, d, 0), (d, d, d, 2), (2 * f, f, d, 1), (d, d, f, 2)):
            assert all(plan(lib, T, (N + 255) // 256 * 256, o, K, e, 4096)[0] != 10 for T in range(1, 257, 5)), (name, N, K)
    for d, f in ((256, 704), (512, 1408)):
        for T in (385, 512, 640):
            for N, o, K, e in ((3 * d, 3 * d, d, 0), (d, d, d, 2), (d, d, f, 2)):
                assert plan(lib, T, (N + 255) // 256 * 256, o, K, e, 4096)[0] == 10, (d, T, N, K)


def test_large_batches_do_not_take_64_token_rows_with_loader_waves(lib):
    # beyond 1100 rows a panel of W is read by 18 and more such token tiles, which find it in L2: the form without loader waves (10) measured 3 .. 7 % faster
    # than the one with them (7) for O and down of narrow models
    taken = set()
    for name, (d, f) in WIDTHS.items():
        for N, o, K, e in ((3 * d, 3 * d, d, 0), (d, d, d, 2), (2 * f, f, d, 1), (d, d, f, 2)):
            taken |= {(name, plan(lib, T, (N + 255) // 256 * 256, o, K, e, 4096)[0]) for T in range(1101, 4097, 7)}
    assert all(tile not in (7, 11, 18) for _, tile in taken)
    assert ("tiny", 10) in taken and ("1k", 10) in taken


@pytest.mark.parametrize("T", [129, 147, 160])
def test_no_tile_is_prescribed_for_129_to_160_rows(lib, T):
    # gate/up of 7168 columns: 128 x 160 makes 296 workgroups, a second round for 40 of them; with tiles that go round once a step of 129 rows takes 343 us a layer instead of 356
    N, f = 37888, 18944
    bf, bt = tile_info(lib, plan(lib, T, N, f, 7168, 1, 4096)[0])[1][:2]
    assert -(-N // bf) * -(-T // bt) <= 256, (bf, bt)
    assert tile_info(lib, plan(lib, T, 4096, 4096, 4096, 2, 4096)[0])[1][:2] == (64, 256)      # O of the 7B shape: a step of 150 rows 150.9 -> 149.8 us a layer
