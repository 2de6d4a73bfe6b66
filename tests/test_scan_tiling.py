"""How a long trace is cut into tiles (CPU): on both sides of every limit a tile is one pass of its workgroup where the events
are loaded once, the tiles cover their list, and there are no more of them than a workgroup reads the sums of."""
import ctypes

import pytest

THREADS, MAX_TILES = 256, 1024


def tiling(n_ev, n_pe, n_ops):
    import paper_2509_11076_amd.binding as B
    f = ctypes.CDLL(B.LIB_PATH).ss_scan_tiling
    f.argtypes, f.restype = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_void_p], None
    out = (ctypes.c_uint32 * 5)()
    f(n_ev, n_pe, n_ops, out)
    return list(out)


@pytest.mark.parametrize("n", [0, 1, 2047, 2048, 2049, 4097, 65536, 131071, 131072, 131073, 140000, 262144, 262145, 400000, 524288,
                               524289, 600000, 1048576, 1048577, 1 << 22, (1 << 31) - 4096])
@pytest.mark.parametrize("other", [0, 3, 131073, 300000, 524289, 1048577])
def test_tiles(n, other):
    for n_ops in {0, 1, 2900, 65536, 262144, 300000, 1000000, 1 << 23, min(2 * n, 1 << 23), min(2 * n + 1, 1 << 23)}:
        for lists in ((n, other), (other, n)):
            per_lane, *rest = tiling(*lists, n_ops)
            assert per_lane == (2 if max(lists) <= 524288 else 4 if max(lists) <= 1048576 else 8)
            for events, tile, tiles in zip(lists, rest[::2], rest[1::2]):
                assert tiles == max(1, -(-events // tile)) <= MAX_TILES
                assert per_lane == 8 or tile <= THREADS * per_lane


@pytest.mark.parametrize("n_ev,n_pe,n_ops,few", [
    (100000, 0, 40000, 0), (0, 100000, 40000, 0), (5000, 0, 9000, 0), (0, 0, 9000, 0), (0, 0, 1, 0),         # a list without events has no gaps
    (10, 0, 9000, 1), (0, 10, 9000, 1), (100000, 10, 9000, 1), (1000, 0, 8000, 0), (1000, 0, 8001, 1), (0, 70, 561, 1),
    (100000, 70, 561, 1), (100000, 70, 560, 0), (2049, 0, 1 << 23, 0),      # 8 operators to an event; 8 events to a tile
])
def test_whose_gaps_are_filled_together(n_ev, n_pe, n_ops, few):
    import paper_2509_11076_amd.binding as B
    f = ctypes.CDLL(B.LIB_PATH).ss_scan_few_events
    f.argtypes, f.restype = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32], ctypes.c_int
    assert f(n_ev, n_pe, n_ops) == few
