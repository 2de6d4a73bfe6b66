"""Host calls return once their last kernel has told the host, or, where that takes long, once the stream is idle: the same
results on an idle GPU and beside products that hold every compute unit, many calls in a row, buffers growing in between."""
import numpy as np
import pytest

from test_gpu_trace_scan_match import P, ctx          # noqa: F401  (fixtures)
from test_gpu_scan_edges import events

pytestmark = pytest.mark.gpu


def operators(P, rng, n):                              # noqa: F811
    ops = np.zeros(n, dtype=P.OP_DT)
    ops["op_token"], ops["stack_hash"], ops["n_out"] = rng.integers(1, 9, n), rng.integers(1, 5, n), 1
    ops["sig"] = 1 | (1 << 8)
    return ops


def test_results_beside_work_on_the_compute_stream(P, ctx):                          # noqa: F811
    import torch
    rng = np.random.default_rng(11)
    calls = []
    for n_ev, n_ops in ((100, 66), (9000, 3000), (60000, 9000), (300, 200)):
        ev, pe = events(rng, n_ev, n_ops), events(rng, n_ev // 4, n_ops)
        calls.append(lambda ev=ev, pe=pe, n=n_ops: P.ss_timeline_scan(ctx, ev, pe, n, 5, 1 << 40, want_timeline=True))
        calls.append(lambda ev=ev, pe=pe, n=n_ops: P.ss_timeline_scan_batch(ctx, ev, [pe, None, pe[:50]], n, 5, 9, want_per_op=True))
    for n, k in ((90, 30), (1500, 400), (7000, 5000)):
        ref, cur = operators(P, rng, n), operators(P, rng, n + 7)
        anchors = np.zeros(k, dtype=P.ANCHOR_DT)
        anchors["ref_op"] = np.sort(rng.choice(n, k, replace=False))
        for flags in (0, P.SS_MATCH_HISTOGRAM, P.SS_MATCH_ALIGN):
            calls.append(lambda r=ref, c=cur, a=anchors, f=flags: P.ss_match_sequence(ctx, r, c, a, flags=f))
        calls.append(lambda r=ref, c=cur: P.ss_match_sequence(ctx, r, c, None))
        calls.append(lambda r=ref, c=cur, a=anchors: P.ss_align_sequence(ctx, r, c, a))

    def same(x, y):
        if isinstance(x, list):
            return len(x) == len(y) and all(same(p, q) for p, q in zip(x, y))
        return x.keys() == y.keys() and all(np.array_equal(x[k], y[k]) for k in x)
    idle = [f() for f in calls]
    m = torch.ones(8192, 8192, dtype=torch.bfloat16, device="cuda")
    for _ in range(2):
        for f, want in zip(calls, idle):
            for _ in range(3):
                m @ m                                  # about a millisecond each
            assert same(f(), want)
        torch.cuda.synchronize()
        for f, want in zip(calls, idle):
            assert all(same(f(), want) for _ in range(5))


def in_turn(call, want):
    """two inputs in turn, so that a result that is late is the other input's; beside short products and beside kernels that
    keep the caches full of their own stores (a word that did not wait for other dies' results: 2 to 4 % of the calls)"""
    import torch
    m = torch.ones(4096, 4096, dtype=torch.bfloat16, device="cuda")
    full = torch.zeros(1 << 28, dtype=torch.uint8, device="cuda")
    for work in (lambda: m @ m, lambda: full.add_(1)):
        for _ in range(250):
            for _ in range(6):
                work()
            for i in (0, 1):
                got = call(i)
                assert all(np.array_equal(got[k], want[i][k]) for k in got)
        torch.cuda.synchronize()


@pytest.mark.parametrize("n_ev,n_ops", [(60000, 9000), (20000, 3000)])
def test_the_word_comes_after_every_result(P, ctx, n_ev, n_ops):                     # noqa: F811
    rng = np.random.default_rng([n_ev, n_ops])
    inputs = [(events(rng, n_ev, n_ops), events(rng, n_ev // 4, n_ops), 5 + 1000003 * i) for i in (1, 2)]

    def call(i):
        ev, pe, base = inputs[i]
        return P.ss_timeline_scan(ctx, ev, pe, n_ops, base, 1 << 40, want_timeline=True)
    in_turn(call, [call(0), call(1)])


@pytest.mark.parametrize("what,n,k", [
    ("match", 1500, 400), ("match", 7000, 5000), ("match", 40000, 300),      # searches in registers, by numbers; sums of many workgroups
    ("match", 60000, 0), ("histogram", 9000, 0), ("histogram", 9000, 900),   # the sums alone
    ("align", 1500, 40), ("align", 3000, 40), ("align", 7000, 40),           # one launch; rows walked by the host; pairs from the GPU
])
def test_the_word_comes_after_every_result_of_earlier_kernels(P, ctx, what, n, k):   # noqa: F811
    """the sums of the cosine are written by the first kernel of a call, an aligner's pairs partly by the one before the last;
    expected values from the oracle"""
    import oracle
    rng = np.random.default_rng([n, k])
    inputs = []
    for extra in (3, 11):
        ref, cur = operators(P, rng, n), operators(P, rng, n + extra)
        anchors = np.zeros(k, dtype=P.ANCHOR_DT)
        anchors["ref_op"] = np.sort(rng.choice(n, k, replace=False))
        inputs.append((ref, cur, anchors))

    def call(i):
        if what == "align":
            return P.ss_align_sequence(ctx, *inputs[i])
        return P.ss_match_sequence(ctx, *inputs[i], flags=P.SS_MATCH_HISTOGRAM if what == "histogram" else 0)
    want = [call(0), call(1)]
    for (ref, cur, _), got in zip(inputs, want):
        if what != "align":
            a, b = cur["op_token"].astype(np.int64), ref["op_token"].astype(np.int64)
            if what == "histogram":
                a, b = np.bincount(a, minlength=64), np.bincount(b, minlength=64)
            b = np.pad(b, (0, len(a) - len(b)))
            assert (got["dot"], got["na"], got["nb"]) == ((a * b).sum(), (a * a).sum(), (b * b).sum())
        elif n <= 1500:
            ora = oracle.align_anchors(oracle.ops_tuples(ref), oracle.ops_tuples(cur), [])
            assert np.array_equal(got["ref_to_cur"], ora["ref_to_cur"])
    in_turn(call, want)


@pytest.mark.parametrize("n", [1500, 2500, 3000, 7000, 20000])
def test_words_of_an_aligners_first_kernels(P, ctx, n):                              # noqa: F811
    """the number of keys and, in aligned matching, the cosine's sums are pinned by the first kernels, of up to 80 workgroups, and the
    host waits for the last one, of one to 313: inputs of different keys and tokens in turn"""
    rng = np.random.default_rng([n, 5])
    inputs, want = [], [[], []]
    for stacks, token in ((3, 0), (7, 900)):
        ref, cur = operators(P, rng, n), operators(P, rng, n + 30)
        for ops in (ref, cur):
            ops["op_token"] += token
            ops["stack_hash"] = rng.integers(0, stacks, len(ops))
        anchors = np.zeros(40, dtype=P.ANCHOR_DT)
        anchors["ref_op"] = np.sort(rng.choice(n, 40, replace=False))
        inputs.append((ref, cur, anchors))

    def aligned(i):
        r = P.ss_align_sequence(ctx, *inputs[i])
        return {k: r[k] for k in ("n_keys", "lcs", "ref_to_cur", "new_idx")}

    def matched(i):
        r = P.ss_match_sequence(ctx, *inputs[i], flags=P.SS_MATCH_ALIGN)
        return {k: r[k] for k in ("dot", "na", "nb", "new_idx", "level")}
    for i, (ref, cur, _) in enumerate(inputs):
        a, b = cur["op_token"].astype(np.int64), np.pad(ref["op_token"].astype(np.int64), (0, 30))
        want[0].append(dict(aligned(i), n_keys=len(np.unique(cur[["op_token", "stack_hash", "sig"]]))))
        want[1].append(dict(matched(i), dot=(a * b).sum(), na=(a * a).sum(), nb=(b * b).sum()))
    in_turn(aligned, want[0])
    in_turn(matched, want[1])


@pytest.mark.parametrize("n_ev,n_pe,n_ops", [(1000, 400, 9000), (9000, 3000, 6000), (60000, 20, 30000)])
def test_lists_out_of_order_in_turn(P, ctx, n_ev, n_pe, n_ops):                      # noqa: F811
    """the sums that other workgroups gathered are there for the one that does the operators"""
    import oracle
    rng = np.random.default_rng([n_ev, n_ops, 9])
    inputs, want = [], []
    for base in (5, 1 << 50):
        ev, pe = events(rng, n_ev, n_ops), events(rng, n_pe, n_ops)
        ora = oracle.timeline_scan(ev, pe, n_ops, base, 1 << 40)
        inputs.append((ev[rng.permutation(n_ev)], pe[::-1].copy(), base))
        want.append(dict(per_op=ora["per_op"], mre=ora["mre"], peak=ora["peak"], argpeak_op=ora["argpeak_op"], final=ora["final"]))

    def call(i):
        ev, pe, base = inputs[i]
        r = P.ss_timeline_scan(ctx, ev, pe, n_ops, base, 1 << 40)
        return {k: r[k] for k in want[i]}
    in_turn(call, want)
