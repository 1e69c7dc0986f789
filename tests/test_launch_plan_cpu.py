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
