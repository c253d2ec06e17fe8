"""Which attention kernel a pass takes and in which shape: the library's own rule, compiled for the host."""
import collections
import ctypes as C
import itertools

import pytest

from tests.launch_rules import rules

Launch = collections.namedtuple("Launch", "small nwv ksplit row_groups chunk_blocks chunks")


def launch(D, Hkv, group, M, P, max_chunks=64):
    out = (C.c_int * 6)()
    rules().attention(D, Hkv, group, M, P, int(M > 80), 8 if M > 80 else max_chunks, out)
    return Launch(*out)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hkv,group", [(1, 1), (1, 4), (2, 16), (3, 1), (4, 7), (8, 4), (8, 8), (32, 1), (40, 1), (64, 8), (96, 1), (97, 1), (256, 1), (512, 1)])
def test_every_launch_holds_its_work(D, Hkv, group):
    for M, P in itertools.product([1, 2, 4, 8, 15, 16, 17, 24, 33, 48, 64, 65, 80, 81, 200, 333, 1024],
                                  [0, 1, 31, 60, 100, 127, 128, 250, 500, 639, 640, 700, 1000, 1023, 1024, 1025, 2047, 4096, 8192, 40000]):
        a, NB, tiles = launch(D, Hkv, group, M, P), (P + M + 31) // 32, (M * group + 15) // 16
        assert a.chunks <= (8 if M > 80 else 64) and (a.chunks - 1) * a.chunk_blocks < NB <= a.chunks * a.chunk_blocks
        if a.small:
            assert tiles == 1 and NB <= 32 and a.chunks == 1 and a.row_groups == 1
            continue
        assert (a.nwv, a.ksplit) in {(4, 2), (8, 2), (10, 2), (8, 1)}
        assert (a.row_groups - 1) * (a.nwv // a.ksplit) < tiles <= a.row_groups * (a.nwv // a.ksplit)
        # four waves: the first two stages are requested without a look at the row group's own number of blocks
        assert a.nwv != 4 or a.row_groups == 1


# The sides of the rule's lines where one form was measured against the other, whole layers (kernel and merge, us, on either side in the rule's comments)
@pytest.mark.parametrize("Hkv,group,M,P,small", [(32, 1, 8, 632, True), (32, 1, 8, 633, False), (64, 1, 8, 700, False), (96, 1, 8, 760, True), (96, 1, 8, 761, False), (97, 1, 8, 800, True), (128, 1, 8, 1016, True),
                                                 (128, 1, 8, 1017, False), (256, 1, 16, 900, True), (8, 4, 4, 636, True), (8, 4, 4, 637, False)])
def test_one_tile_without_a_loop(Hkv, group, M, P, small):
    assert launch(128, Hkv, group, M, P).small == small
    assert launch(64, Hkv, group, M, P).small == (P + M <= 1024)


@pytest.mark.parametrize("Hkv,group,M", [(1, 1, 8), (2, 4, 4), (2, 4, 16), (4, 1, 8), (2, 4, 64), (12, 1, 8), (8, 4, 16)])
@pytest.mark.parametrize("P,most", [(1100, 12), (1400, 12), (2000, 12), (3000, 15), (5000, 19), (8200, 24), (16300, 34)])
def test_few_heads_leave_the_merge_few_chunks(Hkv, group, M, P, most):
    for D in (64, 128):
        assert min(6, 256 // Hkv) <= launch(D, Hkv, group, M, P).chunks <= most


@pytest.mark.parametrize("P,most", [(900, 16), (1400, 16), (4000, 23), (8200, 33)])
def test_few_heads_of_one_team(P, most):
    assert 8 <= launch(64, 2, 4, 24, P).chunks <= most and 8 <= launch(128, 8, 4, 32, P).chunks <= most


@pytest.mark.parametrize("D,Hkv,group,M,P,one", [
    (128, 8, 4, 16, 100, True), (128, 8, 4, 16, 200, False), (128, 8, 4, 16, 250, False), (128, 32, 4, 16, 180, True), (128, 32, 4, 16, 200, False),
    (128, 1, 1, 64, 100, True), (128, 1, 1, 64, 200, False), (128, 32, 1, 64, 250, True), (128, 40, 1, 64, 250, True), (128, 40, 1, 64, 260, False),
    (128, 1, 4, 64, 20, False), (128, 8, 4, 64, 100, True), (128, 8, 4, 64, 200, False), (128, 32, 4, 64, 230, True),
    (128, 8, 4, 32, 60, False), (128, 8, 4, 32, 20, True), (128, 64, 8, 16, 90, True), (128, 32, 1, 80, 60, True), (128, 1, 1, 80, 60, False),
    (64, 8, 4, 16, 200, True), (64, 8, 4, 16, 250, False), (64, 1, 4, 64, 100, True), (64, 1, 4, 64, 200, False), (64, 8, 4, 32, 90, True)])
def test_short_context_in_one_chunk_or_more(D, Hkv, group, M, P, one):
    assert (launch(D, Hkv, group, M, P).chunks == 1) == one
