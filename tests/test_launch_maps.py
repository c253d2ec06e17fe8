"""The maps from workgroups to rows and tiles that put writers of one cache line on one die, the library's own, compiled for the host: every
row (times column range) and every tile has exactly one workgroup, whatever the counts, and the rows of a line share a die."""
import ctypes as C

import pytest

from tests.launch_rules import rules


def row_units(M, parts):
    """RowUnits: {workgroup: (row, part)} of the workgroups that have one."""
    part, out, log2 = C.c_int(), {}, parts.bit_length() - 1
    for b in range(rules().row_blocks(M, log2)):
        m = rules().row_of(M, log2, b, C.byref(part))
        if m < M:
            out[b] = (m, part.value)
    return out


@pytest.mark.parametrize("parts", [1, 2, 4, 8])
@pytest.mark.parametrize("M", [1, 5, 8, 9, 17, 64, 65, 80, 81, 333, 1000, 1024])
def test_rows(M, parts):
    got = row_units(M, parts)
    assert sorted(got.values()) == [(m, p) for m in range(M) for p in range(parts)]
    die = {}
    for b, (m, p) in got.items():
        assert die.setdefault((m // 8, p), b % 8) == b % 8


@pytest.mark.parametrize("heads", [1, 2, 3, 12, 32, 97])
@pytest.mark.parametrize("M", [1, 5, 8, 9, 17, 64, 80, 81, 1024])
def test_rows_of_heads(M, heads):
    head, got, die = C.c_int(), [], {}
    for b in range(rules().head_blocks(M, heads)):
        m = rules().head_row_of(M, heads, b, C.byref(head))
        if m < M and head.value < heads:
            got.append((m, head.value))
            assert die.setdefault((m // 8, head.value), b % 8) == b % 8
    assert sorted(got) == [(m, h) for m in range(M) for h in range(heads)]


@pytest.mark.parametrize("d", [64, 320, 512, 768, 4096, 5120, 8192])
@pytest.mark.parametrize("M", [1, 32, 33, 80, 81, 1024])
def test_column_ranges(M, d):
    parts = rules().parts_of(M, d)
    assert parts in (1, 2, 4, 8) and d % (64 * parts) == 0


@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 48, 72, 192, 230, 255, 256, 257, 501, 1000, 4096])
def test_tiles(n):
    places = [rules().place(b, n) for b in range(n)]
    assert sorted(places) == list(range(n))
    for die in range(8):
        mine = places[die::8]
        assert mine == list(range(mine[0], mine[0] + len(mine))) if mine else True
