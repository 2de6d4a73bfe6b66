"""GPU parity of the timeline scan where its kernels change form: one workgroup with its tables in LDS (256 or 1,024
lanes), tiles over two launches, lists in and out of operator order, operators without events, empty lists, deltas of
zero.  Exact comparison with the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_trace_scan_match import P, ctx, assert_scan_equal          # noqa: F401  (fixtures)
from test_zz_no_alloc import static_scan

pytestmark = pytest.mark.gpu


def events(rng, n_ev, n_ops, runs=False):
    """n_ev events in operator order; a few deltas are zero; with `runs` most belong to a few operators"""
    op = rng.integers(0, n_ops, n_ev)
    if runs and n_ev:
        few = op[:1 + n_ev // 500]
        op = np.where(rng.random(n_ev) < 0.9, few[rng.integers(0, len(few), n_ev)], op)
    ev = np.zeros(n_ev, dtype=W.EVENT_DT)
    ev["op_idx"] = np.sort(op)
    ev["tensor_id"] = np.arange(n_ev)
    ev["delta"] = rng.integers(-(1 << 40), 1 << 40, n_ev) * (rng.random(n_ev) > 0.05)
    return ev


def both_ways(P, ctx, ev, pe, n_ops, base, budget):               # noqa: F811
    import torch
    ora = oracle.timeline_scan(ev, pe, n_ops, base, budget)
    assert_scan_equal(P.ss_timeline_scan(ctx, ev, pe, n_ops, base, budget, want_timeline=True), ora)
    if len(ev) + len(pe) <= 262144 and n_ops <= 65536:
        got = static_scan(P, torch, ctx, ev, pe, n_ops, base, budget)
        assert got["flags"] == 0
        assert_scan_equal(got, ora)
    return ora


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [
    (1, 0, 1), (0, 1, 3), (63, 1, 5), (64, 64, 64), (1000, 24, 66), (1000, 25, 66),          # 256 lanes | 1,024 lanes
    (255, 257, 2900), (255, 257, 2901),                                                      # LDS tables | device tables
    (4096, 0, 700), (4000, 97, 700), (0, 4097, 700), (2048, 2049, 3000),                     # one launch | two
    (2047, 3000, 40), (6144, 2048, 9000), (40, 7, 60001), (30000, 20000, 1),
    (3000, 2050, 6000), (3000, 2050, 6001), (2049, 2048, 40000), (20000, 3, 65536),          # small tiles where gaps are wide
])
def test_edges_of_the_forms(P, ctx, n_ev, n_pe, n_ops):           # noqa: F811
    rng = np.random.default_rng([n_ev, n_pe, n_ops])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops, runs=True)
    both_ways(P, ctx, ev, pe, n_ops, -7, 1 << 41)


def test_operators_without_events_and_events_of_one_operator(P, ctx):       # noqa: F811
    rng = np.random.default_rng(5)
    for n_ops, at in ((2000, [0, 1999]), (2000, [777]), (40000, [39999]), (40000, [0, 20000])):
        ev = events(rng, 300, len(at))
        ev["op_idx"] = np.asarray(at)[ev["op_idx"]]
        pe = events(rng, 5000 if n_ops > 2900 else 50, 1)
        pe["op_idx"] = at[0]
        both_ways(P, ctx, ev, pe, n_ops, 1 << 45, 0)


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [(700, 200, 66), (3000, 100, 700), (300, 20, 5000), (9000, 4000, 700), (70000, 50, 9000),
                                             (1500, 36, 4000), (1500, 37, 4000)])      # gathered by one workgroup | by all
def test_lists_out_of_order_give_the_same_operators(P, ctx, n_ev, n_pe, n_ops):      # noqa: F811
    import torch
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 1])
    ev, pe = events(rng, n_ev, n_ops, runs=True), events(rng, n_pe, n_ops)
    ora = oracle.timeline_scan(ev, pe, n_ops, 11, 1 << 40)
    for a, b in ((ev[rng.permutation(n_ev)], pe), (ev, pe[::-1].copy()), (np.roll(ev, 1), pe)):
        lib = P.ss_timeline_scan(ctx, a, b, n_ops, 11, 1 << 40)
        assert_scan_equal(lib, ora, timeline=False)
        assert lib["sorted"] == 0
        got = static_scan(P, torch, ctx, a, b, n_ops, 11, 1 << 40)
        assert got["flags"] == 2
        assert_scan_equal(got, ora, timeline=False)
        with pytest.raises(P.SsError) as e:
            P.ss_timeline_scan(ctx, a, b, n_ops, 11, 1 << 40, want_timeline=True)
        assert e.value.code == P.SS_E_ORDER
        one = P.ss_timeline_scan_batch(ctx, a, [b, None], n_ops, 11, 1 << 40, want_per_op=True)
        assert one[0]["peak"] == ora["peak"] and np.array_equal(one[0]["per_op"], ora["per_op"])
        bad = a.copy()
        bad["op_idx"][n_ev // 2] = n_ops
        with pytest.raises(P.SsError) as e:
            P.ss_timeline_scan(ctx, bad, b, n_ops, 11, 1 << 40)
        assert e.value.code == P.SS_E_INVAL


@pytest.mark.parametrize("n_ev,n_ops", [(500, 66), (9000, 2900), (9000, 2901), (40, 40000)])
def test_batch_with_tables_in_lds_and_in_device_memory(P, ctx, n_ev, n_ops):         # noqa: F811
    rng = np.random.default_rng([n_ev, n_ops])
    ev = events(rng, n_ev, n_ops)
    cands = [None, events(rng, 1, n_ops), events(rng, 4100, n_ops), events(rng, 64, n_ops, runs=True)]
    lib = P.ss_timeline_scan_batch(ctx, ev, cands, n_ops, 3, 1 << 40, want_per_op=True)
    for r, c in zip(lib, cands):
        ora = oracle.timeline_scan(ev, c, n_ops, 3, 1 << 40)
        assert (r["peak"], r["argpeak_op"], r["n_over"], r["final"]) == (ora["peak"], ora["argpeak_op"], ora["n_over"], ora["final"])
        assert np.array_equal(r["per_op"], ora["per_op"])


@pytest.mark.parametrize("n_ops", [700, 5000])
def test_batch_lists_out_of_order_from_the_start_or_late(P, ctx, n_ops):             # noqa: F811
    """several passes over the events: what is out of order shows in the first, at an edge or in the last; an operator out
    of range behind it is still found"""
    rng = np.random.default_rng([n_ops, 7])
    ev, pe = events(rng, 9000, n_ops), events(rng, 4200, n_ops)
    ora = oracle.timeline_scan(ev, pe, n_ops, 11, 1 << 40)
    none = oracle.timeline_scan(ev, None, n_ops, 11, 1 << 40)

    def moved(x, where):
        rest = x[:-1] if where < len(x) // 2 else x[1:]
        return np.insert(rest, where, x[-1] if where < len(x) // 2 else x[0])
    for a, b in [(moved(ev, w), pe) for w in (0, 4095, 4096, 8999)] + [(ev, moved(pe, w)) for w in (0, 4199)]:
        lib = P.ss_timeline_scan_batch(ctx, a, [b, None, b], n_ops, 11, 1 << 40, want_per_op=True)
        for r, o in zip(lib, (ora, none, ora)):
            assert (r["peak"], r["argpeak_op"], r["n_over"], r["final"]) == (o["peak"], o["argpeak_op"], o["n_over"], o["final"])
            assert np.array_equal(r["per_op"], o["per_op"])
        for late in (a.copy(), a), (b.copy(), b):
            late[0]["op_idx"][-2] = n_ops
            with pytest.raises(P.SsError) as e:
                P.ss_timeline_scan_batch(ctx, late[0] if late[1] is a else a, [None, late[0] if late[1] is b else b], n_ops, 11, 1 << 40)
            assert e.value.code == P.SS_E_INVAL


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [
    (256, 0, 66), (192, 64, 700), (193, 64, 700), (0, 257, 31), (1024, 0, 32), (768, 256, 33),     # lanes and events to a lane
    (769, 256, 1000), (1792, 255, 90), (1793, 256, 2899), (3840, 256, 2000), (3841, 255, 2000),    # one workgroup | two launches
    (2048, 2048, 2560), (2048, 2048, 2561), (2048, 2048, 2600), (5, 3, 2900), (4090, 1, 2900),     # tables and timeline in LDS
])
def test_one_workgroup_forms(P, ctx, n_ev, n_pe, n_ops):          # noqa: F811
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 4])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops, runs=True)
    ora = both_ways(P, ctx, ev, pe, n_ops, 1 << 44, 9)
    for r, c in zip(P.ss_timeline_scan_batch(ctx, ev, [pe, None, pe[:7]], n_ops, 1 << 44, 9, want_per_op=True), (pe, None, pe[:7])):
        o = ora if c is pe else oracle.timeline_scan(ev, c, n_ops, 1 << 44, 9)
        assert (r["peak"], r["argpeak_op"], r["n_over"], r["final"]) == (o["peak"], o["argpeak_op"], o["n_over"], o["final"])
        assert np.array_equal(r["per_op"], o["per_op"])


def test_every_operator_alike_and_the_lowest_of_equal_peaks(P, ctx):                 # noqa: F811
    for n_ops in (65, 2900, 9000):
        ev = np.zeros(2 * n_ops if n_ops < 2000 else 2000, dtype=W.EVENT_DT)
        ev["op_idx"] = np.arange(len(ev)) % n_ops
        ev["delta"] = np.where(np.arange(len(ev)) % 2 == 0, 7, -7)
        ev = ev[np.argsort(ev["op_idx"], kind="stable")]
        both_ways(P, ctx, ev, np.zeros(0, dtype=W.EVENT_DT), n_ops, -(1 << 62), -(1 << 62) + 3)


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [
    (4096, 513, 700), (4607, 512, 700), (5121, 0, 9),                                # tiles of 512 events and their edges
    (524288, 512, 500), (524289, 1025, 500), (1048576, 0, 40), (1048577, 3, 40),     # two a lane | four | passes of eight
])
def test_tiles_take_up_the_sums_before_them(P, ctx, n_ev, n_pe, n_ops):              # noqa: F811
    """each form with the usual wait for the tiles before, and with none: then a workgroup adds up their events itself"""
    import ctypes
    lib = P._lib
    lib.ss_scan_wait_limit.argtypes, lib.ss_scan_wait_limit.restype = [ctypes.c_void_p, ctypes.c_uint32], None
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 3])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops, runs=True)
    ora = both_ways(P, ctx, ev, pe, n_ops, 5, 1 << 41)
    lib.ss_scan_wait_limit(ctx, 1)
    assert_scan_equal(P.ss_timeline_scan(ctx, ev, pe, n_ops, 5, 1 << 41, want_timeline=True), ora)


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [
    (131072, 0, 262145), (131073, 0, 262147), (0, 131073, 262147), (140000, 140000, 300000), (400000, 9, 1000000),   # two a lane
    (600000, 3, 1300000), (524289, 140000, 300000), (3, 1048577, 2200000),                                          # four | passes
])
def test_more_operators_than_events_and_many_of_both(P, ctx, n_ev, n_pe, n_ops):     # noqa: F811
    """tiles of gaps to be filled that would take more events than a workgroup loads at once; what is wrong with a tile's
    last event is found too"""
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 5])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops, runs=True)
    ora = both_ways(P, ctx, ev, pe, n_ops, 5, 1 << 41)
    assert_scan_equal(P.ss_timeline_scan(ctx, ev, pe, n_ops, 5, 1 << 41), ora, timeline=False)
    lists = [ev, pe]
    which = int(n_pe > n_ev)
    for at in (511, 513, 551, 1023, 1025):                   # with the one before it out of order, or out of range
        swapped = lists[which].copy()
        swapped[[at, at - 1]] = swapped[[at - 1, at]]
        if swapped["op_idx"][at] != swapped["op_idx"][at - 1]:
            one = list(lists)
            one[which] = swapped
            lib = P.ss_timeline_scan(ctx, one[0], one[1], n_ops, 5, 1 << 41)
            assert lib["sorted"] == 0
            assert_scan_equal(lib, ora, timeline=False)
        one = list(lists)
        one[which] = lists[which].copy()
        one[which]["op_idx"][at] = n_ops
        with pytest.raises(P.SsError) as e:
            P.ss_timeline_scan(ctx, one[0], one[1], n_ops, 5, 1 << 41)
        assert e.value.code == P.SS_E_INVAL


@pytest.mark.parametrize("n_ops", [32, 1024, 1025, 2046, 2047, 2048, 2049, 2900])
@pytest.mark.parametrize("at", [(0,), (0.5,), (1,), (0, 1), (0.3, 0.7)])
def test_wide_gaps_in_one_workgroup(P, ctx, n_ops, at):           # noqa: F811
    """a few events of a few operators, far apart, at the ends, beside an empty list and beside one another"""
    rng = np.random.default_rng([n_ops, len(at)])
    places = np.asarray([int(x * (n_ops - 1)) for x in at])
    ev = events(rng, 2 * len(at), len(at))
    ev["op_idx"] = np.sort(places[ev["op_idx"]])
    other = events(rng, 3, n_ops)
    for a, b in ((ev, other[:0]), (other[:0], ev), (ev, other)):
        both_ways(P, ctx, a, b, n_ops, 3, 1 << 40)


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [(1000, 1, 65536), (9000, 8, 40000), (8, 9000, 40000)])
def test_one_list_out_of_order_beside_a_sparse_one(P, ctx, n_ev, n_pe, n_ops):       # noqa: F811
    """gaps needn't be filled then, and whether they are the operators' sums are those of the lists in order"""
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 2])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops)
    ora = oracle.timeline_scan(ev, pe, n_ops, 0, 1 << 40)
    for a, b in ((ev[::-1].copy(), pe), (ev, pe[::-1].copy())):
        assert_scan_equal(P.ss_timeline_scan(ctx, a, b, n_ops, 0, 1 << 40), ora, timeline=False)


def test_the_numbers_of_scans_start_over(P, ctx):                 # noqa: F811
    """words of the board that no scan has written yet hold 0, so no scan has that number"""
    import ctypes
    lib = P._lib
    lib.ss_scan_number.argtypes, lib.ss_scan_number.restype = [ctypes.c_void_p, ctypes.c_uint32], ctypes.c_int
    rng = np.random.default_rng(12)
    assert lib.ss_scan_number(ctx, 0xFFFFFFFE) == 0
    for n_ev in (5000, 40000, 524288, 9000):                 # more tiles from scan to scan
        ev, pe = events(rng, n_ev, 3000), events(rng, 2000, 3000)
        assert_scan_equal(P.ss_timeline_scan(ctx, ev, pe, 3000, 5, 1 << 41, want_timeline=True),
                          oracle.timeline_scan(ev, pe, 3000, 5, 1 << 41))
