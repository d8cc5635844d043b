"""Which rows a partial tile is loaded from (no GPU needed): every key of the sequence from its own, and nothing at or beyond the
length, which a paged cache need not hold even where the block that the last slot is in would."""
import tri_rules as R


def test_rows_of_a_partial_tile():
    lib = R.library()
    for cnt in range(1, 65):
        for rows in (16, 32):
            for first in range(0, 64, rows):
                start, last = lib.tile_first(first, cnt), lib.tile_last(rows, first, cnt)
                assert start // 16 <= first // 16   # a block that has been looked up: the group's own or, past the end, the last key's
                assert 0 <= last < rows and 0 <= start <= start + last < cnt
                for r in range(rows):
                    if first + r < cnt:
                        assert start + min(r, last) == first + r
