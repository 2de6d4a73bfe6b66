"""GPU parity of the timeline scan where the gaps between few events are the work and a workgroup fills each together: one event to a
tile and as many as there may be, gaps before the first and after the last, several events of one operator, one list without any."""
import numpy as np
import pytest

import oracle
from test_gpu_scan_edges import both_ways, events
from test_gpu_trace_scan_match import P, ctx          # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [
    (1, 0, 3000), (0, 1, 3000), (1, 1, 65536), (2, 3, 4097), (8, 9, 2901), (9, 65, 65536), (360, 12, 2901), (500, 13, 26112),
    (257, 512, 65536), (2047, 1, 16377), (2048, 2049, 65536), (4096, 3, 60000), (2047, 300, 1 << 21),
    (128, 40, 16384), (127, 40, 16385), (40, 2048, 65536), (700, 512, 65537), (300, 1878, 29449),
    (1000, 40, 8000), (1000, 40, 8001),                                                # about eight operators to an event
])
def test_few_events_over_many_operators(P, ctx, n_ev, n_pe, n_ops):           # noqa: F811
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 9])
    for end in (False, True):
        ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops, runs=True)
        for x in (ev, pe):
            if len(x):
                x["op_idx"][0 if end else -1] = 0 if end else n_ops - 1
        if not end:
            ev["op_idx"][:len(ev) // 2] = ev["op_idx"][len(ev) // 2:][:1]      # in front nothing, then many of one operator
        both_ways(P, ctx, ev, pe, n_ops, 5, 1 << 41)


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [(2, 0, 3000), (10, 12, 65536), (100, 3, 65536), (300, 40, 30000), (9, 2000, 9000)])
def test_few_events_out_of_order(P, ctx, n_ev, n_pe, n_ops):                 # noqa: F811
    """an inversion in the first tiles, in the last one, everywhere, in the other list; then a scan in order, which finds no traces of it"""
    rng = np.random.default_rng([n_ev, n_pe, n_ops, 10])
    ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops)
    ev["op_idx"][0], ev["op_idx"][-1] = 3, n_ops - 2
    first, last = ev.copy(), ev.copy()
    first["op_idx"][0] = n_ops - 1
    last["op_idx"][-1] = 1
    for x, y in ((first, pe), (last, pe), (ev[rng.permutation(n_ev)], pe), (ev, pe[::-1].copy()), (ev, pe)):
        ora, got = oracle.timeline_scan(x, y, n_ops, 5, 1 << 41), P.ss_timeline_scan(ctx, x, y, n_ops, 5, 1 << 41)
        for what in ("per_op", "mre", "peak", "argpeak_op", "n_over", "final"):
            assert np.array_equal(got[what], ora[what]), what
