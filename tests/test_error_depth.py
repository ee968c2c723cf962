"""The a-priori error bound of the GPU tests against the order of additions written out: no term of a row
may go through more additions than error_depth says, whatever the row's length and place in the sorted order."""
import pytest

from parity import error_depth, group_pieces


def _tree(depths):
    """A balanced tree over eight values (absent ones count as zero and are added all the same)."""
    d = list(depths) + [0] * (8 - len(depths))
    while len(d) > 1:
        d = [max(a, b) + 1 for a, b in zip(d[::2], d[1::2])]
    return d[0]


def _sequence(depths):
    """Values added one after the other: the first goes through all additions that follow."""
    t = depths[0]
    for x in depths[1:]:
        t = max(t, x) + 1
    return t


def _additions(start, count, C):
    """Most additions that a term of a row goes through whose pairs lie at sorted positions
    [start, start + count), fp32 rows."""
    if count <= C:
        return count                                        # the pairs one after the other, dense_in last
    G = C * group_pieces(C)
    end = start + count
    shares = []
    for g in range(start // G, (end - 1) // G + 1):
        pieces = []
        for p in range(g * G, (g + 1) * G, C):
            n = min(end, p + C) - max(start, p)
            if n > 0:
                pieces.append(n - 1)
        shares.append(_sequence(pieces))
    while len(shares) > 1:                                  # sixteen shares at a time, two batches of eight
        shares = [_sequence([0] + [_tree(shares[i + b:i + min(b + 8, 16)]) for b in (0, 8) if shares[i + b:i + b + 8]])
                  for i in range(0, len(shares), 16)]
    return shares[0] + 1


@pytest.mark.parametrize("C", [8, 16, 32])
def test_no_term_goes_through_more_additions_than_the_bound_says(C):
    G = C * group_pieces(C)
    counts = set(range(1, 4 * G)) | {k * G + e for k in (4, 15, 16, 17, 18, 255, 256, 257) for e in (-1, 0, 1, C)}
    for count in sorted(counts):
        starts = range(G) if count <= 4 * G else (0, 1, C - 1, C, G - C, G - 1)
        worst = max(_additions(s, count, C) for s in starts)
        assert worst <= error_depth(count, C) - 1, (C, count)


def test_the_bound_stays_under_the_tolerance_for_the_longest_row():
    for C in (8, 16, 32):
        assert (error_depth(2 ** 31 - 1, C) - 1) * 2.0 ** -24 < 1e-5
