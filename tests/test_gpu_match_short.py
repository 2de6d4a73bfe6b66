"""GPU parity of the matcher where one workgroup takes short sequences: words of the bit maps, the longest sequences and most
anchors, as many keys as fit and one more, the calls after one that didn't fit, anchors of all levels.  Exact comparison."""
import numpy as np
import pytest

import workloads as W
from test_gpu_match_edges import anchors, check, landings, perturbed, sequence
from test_gpu_trace_scan_match import P, ctx          # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,tokens,stacks", [
    (1, 1, 1, 1), (31, 40, 2, 1), (32, 40, 2, 2), (33, 40, 2, 2), (129, 300, 3, 2), (600, 1023, 4, 2), (1100, 1024, 4, 1), (1100, 1025, 4, 1),
    (2047, 2047, 2, 2), (2048, 2048, 2, 2), (2048, 2049, 2, 2), (2049, 2048, 2, 2),
])
def test_sizes(P, ctx, n, k, tokens, stacks):                     # noqa: F811
    rng = np.random.default_rng([n, k])
    ref = sequence(rng, n, tokens, stacks)
    cur, anc = perturbed(rng, ref), anchors(rng, n, k)
    if n >= 129:
        assert set(landings(ref, cur, anc)[1]) == {0, 1, 2, 255}
    check(P, ctx, ref, cur, anc)
    if 1 < n <= 2048:
        check(P, ctx, cur, ref, anc)                              # the longer one second


@pytest.mark.parametrize("n,keys", [(160, 255), (160, 256), (160, 257), (2048, 48), (2048, 49)])
def test_as_many_keys_as_fit(P, ctx, n, keys):                    # noqa: F811
    rng = np.random.default_rng([n, keys])
    few, many = (np.concatenate([np.arange(c), rng.integers(0, c, 2 * n - c)]) for c in (5, keys))
    anc = anchors(rng, n, 100)
    for key in (many, few, many):                                 # after one that doesn't fit the next calls don't try
        ops = np.zeros(2 * n, dtype=W.OP_DT)
        ops["op_token"] = 1 + key % 7
        ops["stack_hash"] = key // 14
        ops["sig"] = 0x101 + (key // 7 % 2 << 16)
        ops["n_out"] = 2
        check(P, ctx, ops[:n], ops[n:], anc)
        for _ in range(40):
            r = P.ss_match_sequence(ctx, ops[:n], ops[n:], anc)
        idx, lvl = landings(ops[:n], ops[n:], anc)
        assert np.array_equal(r["new_idx"], idx) and np.array_equal(r["level"], lvl)


def test_tokens_out_of_range(P, ctx):                             # noqa: F811
    ops = np.zeros(70, dtype=W.OP_DT)
    ops["op_token"], ops["n_out"] = (1 << 18) - 1, 1
    anc = np.zeros(3, dtype=W.ANCHOR_DT)
    anc["ref_op"] = [0, 69, 70]
    check(P, ctx, ops, ops[:69], anc)
    for at in (0, 69):
        bad = ops.copy()
        bad["op_token"][at] = 1 << 18
        for pair in ((bad, ops), (ops, bad)):
            with pytest.raises(P.SsError):
                P.ss_match_sequence(ctx, *pair, anc)


@pytest.mark.parametrize("n,wrong", [(2048, slice(0, 64)), (2048, slice(64, 128)), (2048, slice(960, 1024)), (2048, slice(0, 1024))])
def test_tokens_out_of_range_whose_squares_wrap_to_zero(P, ctx, n, wrong):         # noqa: F811
    """2^31 four times, at places i and i + 1,024 of both sequences, has squares that add up to 2^64: for one wavefront or all"""
    ref = np.zeros(n, dtype=W.OP_DT)
    ref["op_token"], ref["n_out"] = 1 + np.arange(n) % 7, 1
    cur = ref.copy()
    cur["stack_hash"][5] = 9                                      # the same sequence twice is another path
    anc = np.zeros(3, dtype=W.ANCHOR_DT)
    check(P, ctx, ref, cur, anc)
    for ops in (ref, cur):
        ops["op_token"][:1024][wrong] = ops["op_token"][1024:][wrong] = 1 << 31
    with pytest.raises(P.SsError) as e:
        P.ss_match_sequence(ctx, ref, cur, anc)
    assert e.value.code == P.SS_E_INVAL


@pytest.mark.parametrize("n,k,limit", [(160, 767, 120), (300, 4, 120), (160, 768, 180), (300, 1279, 180), (160, 1280, 256), (300, 2048, 227),
                                       (1156, 480, 75), (1156, 2048, 75), (2048, 100, 48)])
def test_keys_about_what_one_workgroup_takes(P, n, k, limit):              # noqa: F811
    """as many keys as fit LDS and are as fast there, one less and one more, on a context of their own each"""
    rng = np.random.default_rng([n, k])
    anc = anchors(rng, n, k)
    for keys in (limit - 1, limit, limit + 1):
        key = np.concatenate([np.arange(keys), rng.integers(0, keys, 2 * n - keys)])
        rng.shuffle(key)
        ops = np.zeros(2 * n, dtype=W.OP_DT)
        ops["op_token"], ops["stack_hash"], ops["sig"], ops["n_out"] = 1 + key % 7, key // 14, 0x101 + (key // 7 % 2 << 16), 2
        c = P.ss_create(P.ss_config_default())
        try:
            idx, lvl = landings(ops[:n], ops[n:], anc)
            for _ in range(3):
                r = P.ss_match_sequence(c, ops[:n], ops[n:], anc)
                assert np.array_equal(r["new_idx"], idx) and np.array_equal(r["level"], lvl)
        finally:
            P.ss_destroy(c)


def test_contexts_that_begin_with_many_keys(P):                            # noqa: F811
    """some operators are looked at before one workgroup is tried: few keys in those and many in all, many in both, few in both, in any
    order on one context, past the number of calls that aren't tried"""
    rng = np.random.default_rng(41)
    n = 2000

    def ops(key):
        o = np.zeros(len(key), dtype=W.OP_DT)
        o["op_token"], o["stack_hash"], o["sig"], o["n_out"] = 1 + key % 50, key // 100, 0x101 + (key // 50 % 2 << 16), 1
        return o
    anc = anchors(rng, n, 300)
    hidden = np.zeros(n, dtype=np.int64)
    hidden[1::8] = 1 + np.arange(len(hidden[1::8]))                # not among every eighth operator
    forms = [hidden, rng.integers(0, 900, n), rng.integers(0, 30, n), np.arange(n)]
    pairs = [(ops(f), ops(np.roll(f, 5))) for f in forms]
    want = [landings(ref, cur, anc) for ref, cur in pairs]
    small = tuple(x[:40].copy() for x in pairs[2])
    small_want = landings(*small, anc[:9])
    for first in range(4):
        c = P.ss_create(P.ss_config_default())
        try:
            for i in [first] + [x for x in (0, 2, 1, 2, 3, 0) for _ in range(1 if x != 1 else 70)]:
                r = P.ss_match_sequence(c, *pairs[i], anc)
                assert np.array_equal(r["new_idx"], want[i][0]) and np.array_equal(r["level"], want[i][1])
                if i in (1, 2):                                    # sequences much shorter in between
                    r = P.ss_match_sequence(c, *small, anc[:9])
                    assert np.array_equal(r["new_idx"], small_want[0])
        finally:
            P.ss_destroy(c)
