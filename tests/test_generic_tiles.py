"""Tiles of the score kernel for fp32 keys and small blocks, seen without a GPU: 128 keys per workgroup where tiles of 256 would leave
compute units without work, a few with twice the others', or a longer last round; 256 elsewhere, and where the moments of so many
tiles have no room."""
import pytest

import launch_probe


@pytest.mark.parametrize("n,kv_heads,group,parts", [(4096, 1, 4, 1), (65536, 1, 8, 1), (81920, 1, 8, 1), (81921, 1, 8, 2),
                                                    (131072, 1, 8, 2), (98304, 1, 4, 2), (98304, 1, 2, 1), (98305, 1, 2, 2), (131072, 1, 1, 2),
                                                    (8192, 8, 4, 1), (10240, 8, 4, 1), (10241, 8, 4, 2), (16384, 8, 4, 2), (2176, 56, 4, 2),
                                                    (2934, 48, 4, 1), (1100, 128, 4, 1), (1100, 128, 8, 2), (1100, 200, 4, 2), (256, 256, 1, 1),
                                                    (256, 384, 1, 1), (256, 385, 1, 2)])
@pytest.mark.parametrize("entry", ["score", "step"])
def test_keys_per_workgroup(entry, n, kv_heads, group, parts):
    [(status, launches, _)] = launch_probe.run([dict(entry=entry, n=n, kv_heads=kv_heads, group=group, dtype=0)])
    assert status == 0
    [grid] = [grid for name, grid, *_ in launches if "12score_kernel" in name]
    assert grid == (-(-n // (128 * parts)), kv_heads, 1)
