"""The rules by which the score kernels cut a batch into work items and by which a batch gets its kernel (no GPU needed)."""
import random

import pytest

import bench
import tri_rules as R

CUS = 256


@pytest.mark.parametrize("instances,n", [(32, 65536), (16, 131072), (64, 32768), (128, 16384), (256, 8192), (512, 8192)])
def test_whole_items_do_not_make_a_batch_large(instances, n):
    """Batches far below eight items per CU whose cost model ends at 8192 keys: up to four query heads per KV head they stay on
    the kernel that takes every other small batch; above that they keep the sixteen-lane one, the slower of the two, whose sums are nearer to 64 bits
    on short dense sequences."""
    assert R.item_keys(instances, n, CUS) == 8192 and not R.large_batch(instances, n, CUS)
    for group in (1, 2, 3, 4):
        assert not R.sixteen_lane_kernel(group, instances, n, CUS)
    for group in (5, 6, 7, 8):
        assert R.sixteen_lane_kernel(group, instances, n, CUS)


@pytest.mark.parametrize("group,instances,n,expected", [(4, 2048, 8192, True), (4, 2048, 8193, False), (4, 2047, 8192, False),
                                                        (4, 2048, 300, True), (8, 2048, 8193, True), (8, 40, 3000, False)])
def test_where_the_lines_lie(group, instances, n, expected):
    assert R.sixteen_lane_kernel(group, instances, n, CUS) == expected
    for other in (dict(half_split=True), dict(paged=False), dict(rotated=True)):
        assert not R.sixteen_lane_kernel(group, instances, n, CUS, **other)


def test_items():
    rng = random.Random(3)
    for _ in range(3000):
        n, instances = int(2 ** rng.uniform(0, 20)), int(2 ** rng.uniform(0, 14))
        keys = R.item_keys(instances, n, CUS)
        assert 512 <= keys <= 8192 and keys % 64 == 0   # whole tiles, never below what the work list is sized for
        if R.large_batch(instances, n, CUS):
            assert keys == 8192


def test_the_benchmark_names_the_kernel_that_runs():
    rng = random.Random(5)
    for _ in range(3000):
        n, instances, group = int(2 ** rng.uniform(0, 18)), int(2 ** rng.uniform(0, 14)), rng.randint(1, 8)
        half, paged, rotated = (rng.random() < p for p in (0.2, 0.8, 0.2))
        sixteen = R.sixteen_lane_kernel(group, instances, n, CUS, half, paged, rotated)
        assert bench.score_kernel_name(group, instances, n, CUS, True, half, paged, rotated) == \
            ("score_mfma_kernel" if sixteen else "score_lane_kernel"), (group, instances, n, half, paged, rotated)
    assert bench.score_kernel_name(4, 288, 2176, CUS, False, False, False, False) == "score_kernel"
