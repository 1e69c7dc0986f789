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
