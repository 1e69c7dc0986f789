"""The launch plans of the projection products (host queries, no GPU): what
they must guarantee beyond being fast."""

import random

import pytest

from paper_2408_03505_amd import binding as B


def _ceil(a, b):
    return -(-a // b)


def _weight_gradients(count=4000):
    """(tokens, N, K) of random weight gradients, and the smallest and largest
    of the ones that split."""
    rng = random.Random(5)
    cases = [(1024, 8, 8), (1024, 2048, 2048), (16384, 4096, 1024), (8224, 192, 192), (4096, 1024, 1024),
             (2936, 3200, 560), (6304, 768, 768), (1576, 768, 3072)]
    for _ in range(count):
        cases.append((rng.randint(1024, 8224), 8 * rng.randint(1, 512), 8 * rng.randint(1, 512)))
    return cases


def test_weight_gradient_splits_are_no_longer_than_two_128x128_workgroups_per_cu():
    # fp32 results: the length of a split bounds the error of its sums
    splits = 0
    for M, N, K in _weight_gradients():
        sp = B.linear_plan(B.LAYOUT_WGRAD, M, N, K)[2]
        if sp == 1:
            continue
        splits += 1
        s = min(512 // (_ceil(N, 128) * _ceil(K, 128)), M // 512, 16)
        assert s >= 2
        longest = _ceil(_ceil(M, s), 64) * 64
        assert _ceil(_ceil(M, sp), 64) * 64 <= longest, (M, N, K, sp, s)
    assert splits > 500


# Products that a fitted cost table sent to a tile 7 to 27% slower than the
# 128x128, 256x192 and 256x256 tiles of the earlier kernels: several rounds of
# 64x64 tiles over a few k-steps, and weight gradients of few tokens on tiles
# that are alone on their CU.
@pytest.mark.parametrize("layout,M,N,K,slow", [
    (B.LAYOUT_DGRAD, 6563, 832, 192, {(64, 64)}),
    (B.LAYOUT_DGRAD, 5142, 832, 256, {(64, 64), (256, 256)}),
    (B.LAYOUT_FWD, 6345, 896, 256, {(64, 64), (256, 256)}),
    (B.LAYOUT_FWD, 4660, 1216, 256, {(64, 64), (256, 256)}),
    (B.LAYOUT_WGRAD, 381, 2368, 4288, {(64, 64), (256, 256)}),
    (B.LAYOUT_WGRAD, 588, 2560, 14208, {(256, 192), (256, 256)}),
    (B.LAYOUT_WGRAD, 306, 4480, 23488, {(256, 192), (256, 256)}),
    (B.LAYOUT_WGRAD, 65, 18304, 6016, {(256, 192), (256, 256)})])
def test_short_contractions_avoid_the_tiles_that_slowed_them(layout, M, N, K, slow):
    assert B.linear_plan(layout, M, N, K)[:2] not in slow


def test_weight_gradients_over_ten_steps_or_less_run_two_workgroups_to_a_cu():
    rng = random.Random(6)
    for _ in range(2000):
        M, N, K = rng.randint(1, 640), 8 * rng.randint(1, 1024), 8 * rng.randint(1, 1024)
        assert B.linear_plan(B.LAYOUT_WGRAD, M, N, K)[:2] in {(192, 128), (128, 128), (64, 128), (64, 64)}, (M, N, K)


def test_gelu_products_have_plans_of_their_own():
    # ViT-Base: 256x192 tiles for the plain MLP-up product, 128x128 with the
    # GELU epilogue; splits and the register-staged kernel's tiles are shared
    assert B.linear_plan(B.LAYOUT_FWD, 6304, 3072, 768) == (256, 192, 1)
    assert B.linear_plan(B.LAYOUT_FWD_GELU, 6304, 3072, 768) == (128, 128, 1)
    pairs = ((B.LAYOUT_FWD, B.LAYOUT_FWD_GELU), (B.LAYOUT_DGRAD, B.LAYOUT_DGRAD_GELU))
    rng = random.Random(8)
    differ = 0
    for _ in range(1000):
        M, N, K = rng.randint(1, 8224), 8 * rng.randint(1, 1024), rng.choice((8, 64)) * rng.randint(1, 96)
        for plain, gelu in pairs:
            a, b = B.linear_plan(plain, M, N, K), B.linear_plan(gelu, M, N, K)
            assert a[2] == b[2] and (a == b or (a[2] == 1 and K % 64 == 0)), (M, N, K)
            differ += a != b
    assert differ > 50
    for layout in (-1, 5):
        with pytest.raises(B.EncError):
            B.linear_plan(layout, 64, 64, 64)


def test_fetch_floors_are_those_of_the_tiles_that_run():
    import bench
    from paper_2408_03505_amd.synthetic import CONFIGS
    cfg = CONFIGS["vit_base"]
    floors = bench.gemm_fetch_floors(cfg)
    M, H, F = cfg["batch"] * cfg["seq"], cfg["hidden"], cfg["mlp"]
    for n, layout in (("mlp_up_fwd", B.LAYOUT_FWD_GELU), ("mlp_down_bwd_data", B.LAYOUT_DGRAD_GELU)):
        assert floors[n] == bench.fetch_floor(M, F, H, *B.linear_plan(layout, M, F, H)), n
    # a contraction that is no multiple of 64: the register-staged kernel walks
    # its 128x128 tiles in groups of 4 rows, not 8
    odd = dict(cfg, hidden=3080, seq=256, batch=16)
    assert bench.gemm_fetch_floors(odd)["mlp_up_fwd"] == bench.fetch_floor(4096, F, 3080, 128, 128, 1, staged=True)
    assert bench.fetch_floor(4096, F, 3080, 128, 128, 1, staged=True) != bench.fetch_floor(4096, F, 3080, 128, 128, 1)


@pytest.mark.parametrize("gm", (4, 8))
@pytest.mark.parametrize("tm,tn", [(8, 96), (16, 72), (32, 24), (24, 32), (18, 4), (9, 5), (1, 1)])
def test_tile_orders_cover_every_tile_once(tm, tn, gm):
    import bench
    nb = tm * tn
    assert sorted(bench._tile_of(p, nb, tm, tn, gm) for p in range(nb)) == [(a, b) for a in range(tm) for b in range(tn)]


def test_narrow_products_never_run_256_row_tiles():
    # the 256-row kernels' second half tiles start up to 64 rows into an operand
    for layout in range(5):
        for narrow in (8, 24, 40, 56, 64):
            for wide in (8, 256, 4096, 49152, 65536, 131072):
                for k in (64, 1024, 8192, 16320):
                    if wide * k >= 2 ** 31:
                        continue
                    for rows, cols in ((narrow, wide), (wide, narrow)):
                        # a weight gradient's output is [N, K] over M tokens
                        args = (k, rows, cols) if layout == B.LAYOUT_WGRAD else (rows, cols, k)
                        bm, bn, _ = B.linear_plan(layout, *args)
                        assert bm < 256 or (bm, bn) == (256, 128), (layout, rows, cols, k)
