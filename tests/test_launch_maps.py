"""The maps from workgroups to rows and tiles that put writers of one cache line on one die, restated: every row (times column range) and
every tile has exactly one workgroup, whatever the counts, and the rows of a line share a die."""
import pytest


def row_units(M, parts):
    """RowUnits: {workgroup: (row, part)} of the workgroups that have one."""
    blocks = ((M + 7) // 8 * parts + 7) // 8 * 64
    out = {}
    for b in range(blocks):
        unit = b % 8 + b // 64 * 8
        m = unit // parts * 8 + (b >> 3) % 8
        if m < M:
            out[b] = (m, unit % parts)
    return out


@pytest.mark.parametrize("parts", [1, 2, 4, 8])
@pytest.mark.parametrize("M", [1, 5, 8, 9, 17, 64, 65, 80, 81, 333, 1000, 1024])
def test_rows(M, parts):
    got = row_units(M, parts)
    assert sorted(got.values()) == [(m, p) for m in range(M) for p in range(parts)]
    die = {}
    for b, (m, p) in got.items():
        assert die.setdefault((m // 8, p), b % 8) == b % 8


@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 48, 72, 192, 230, 255, 256, 257, 501, 1000, 4096])
def test_tiles(n):
    def place(b):
        die, q, r = b & 7, n >> 3, n & 7
        return die * q + min(die, r) + (b >> 3)
    places = [place(b) for b in range(n)]
    assert sorted(places) == list(range(n))
    for die in range(8):
        mine = places[die::8]
        assert mine == list(range(mine[0], mine[0] + len(mine))) if mine else True
