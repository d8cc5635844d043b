"""Which rows a partial tile is loaded from (no GPU needed): every key of the sequence from its own, and nothing at or beyond the
length, which a paged cache need not hold even where the block that the last slot is in would."""
import tri_rules as R


def test_rows_of_a_partial_tile():
    lib = R.library()
    for cnt in range(1, 65):
        for first in range(0, 64, 16):
            group = lib.tile_group(first, cnt)
            assert group % 16 == 0 and 0 <= group < cnt
            for r in range(16):
                row = lib.tile_row(r, group, cnt)
                assert 0 <= row < 16 and group + row < cnt
                if first + r < cnt:
                    assert group + row == first + r
