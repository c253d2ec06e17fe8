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
