"""GPU parity of the sequence matcher where its kernels change form: a workgroup per anchor, numbered keys, too
many distinct keys for that, inputs through pinned memory or by copy, histograms with tokens in and beyond LDS.  Exact
comparison with the definition in plain Python, itself checked against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import ops_tuples
from test_gpu_trace_scan_match import P, ctx          # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def landings(ref, cur, anchors):
    """per level the operator of the anchor's ordinal among those with its key; the first level whose operator has the
    slot and the data type; the lowest anchor keeps a shared place"""
    keys = (lambda o: (o[0], o[1], o[2]), lambda o: (o[0], o[2]), lambda o: o[0])
    rl, cl = [o.tolist() for o in ref], [o.tolist() for o in cur]
    ordinal, places = [], []
    for key in keys:
        seen, out, at = {}, [], {}
        for o in rl:
            out.append(seen.get(key(o), 0))
            seen[key(o)] = out[-1] + 1
        for j, o in enumerate(cl):
            at.setdefault(key(o), []).append(j)
        ordinal.append(out)
        places.append(at)
    idx, lvl, taken = [], [], set()
    for i, s in anchors.tolist():
        land, level = -1, 255
        if i < len(rl) and rl[i][0]:
            for q, key in enumerate(keys):
                p = places[q].get(key(rl[i]), ())
                if ordinal[q][i] < len(p):
                    j = p[ordinal[q][i]]
                    if s < cl[j][3] and cl[j][2] & 0xFF == rl[i][2] & 0xFF:
                        land, level = j, q
                        break
        if land >= 0 and (land, s) in taken:
            land, level = -1, 255
        taken.add((land, s))
        idx.append(land)
        lvl.append(level)
    return np.array(idx, dtype=np.int32), np.array(lvl, dtype=np.uint8)


def sequence(rng, n, tokens, stacks):
    ops = np.zeros(n, dtype=W.OP_DT)
    ops["op_token"] = rng.integers(1, tokens + 1, n)
    ops["op_token"][rng.random(n) < 0.01] = 0
    ops["stack_hash"] = rng.integers(0, stacks, n) * 0x9E3779B1 & 0xFFFFFFFF
    ops["sig"] = 1 + rng.integers(0, 2, n) + (rng.integers(0, 2, n) << 16)
    ops["n_out"] = rng.integers(0, 3, n)
    return ops


def perturbed(rng, ref):
    cur = ref[rng.random(len(ref)) >= 0.1].copy()
    hit = rng.random(len(cur)) < 0.1
    cur["stack_hash"][hit] ^= 77
    cur["sig"][rng.random(len(cur)) < 0.03] ^= 1 << 16
    return cur


def check(P, ctx, ref, cur, anc):                                 # noqa: F811
    r = P.ss_match_sequence(ctx, ref, cur, anc)
    idx, lvl = landings(ref, cur, anc)
    assert np.array_equal(r["new_idx"], idx) and np.array_equal(r["level"], lvl)
    assert r["n_unmatched"] == int((idx < 0).sum())
    n = max(len(ref), len(cur))
    a, b = (np.pad(x["op_token"].astype(object), (0, n - len(x))) for x in (cur, ref))
    assert (r["dot"], r["na"], r["nb"]) == (int((a * b).sum()), int((a * a).sum()), int((b * b).sum()))


def anchors(rng, n, k):
    anc = np.zeros(k, dtype=W.ANCHOR_DT)
    anc["ref_op"] = rng.integers(0, n + 3, k)                       # some beyond the sequence, many on one operator
    anc["out_slot"] = rng.integers(0, 3, k)
    return anc


def test_the_definition_here_is_the_oracles(P):                   # noqa: F811
    rng = np.random.default_rng(3)
    for n in (1, 40, 200):
        ref = sequence(rng, n, 5, 3)
        cur, anc = perturbed(rng, ref), anchors(rng, n, 50)
        want = oracle.match_anchors(ops_tuples(ref), ops_tuples(cur), anc.tolist())
        got = landings(ref, cur, anc)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("n,k,tokens,stacks", [
    (1, 3, 1, 1), (63, 40, 3, 2), (64, 64, 3, 2), (257, 100, 9, 5), (1030, 300, 12, 9),      # a workgroup per anchor
    (4097, 4000, 12, 9), (9001, 3000, 30, 40),                                               # lists
    (9001, 3000, 200, 1 << 30),                                                              # too many keys for lists
    (140000, 100, 40, 30), (140000, 300, 40, 30),                                            # inputs by copy
    (8192, 2100, 3, 2), (300000, 100, 3, 2),                                                 # whole turns, hits beyond LDS
    (4097, 65537, 12, 9), (9001, 65537, 200, 1 << 30),                                       # many anchors, with lists and without
    (30000, 300, 40, 1 << 30), (9001, 4096, 200, 1 << 30), (9001, 4097, 200, 1 << 30),       # no lists: a workgroup, a wavefront each
    (500, 2047, 12, 9), (500, 2048, 12, 9), (600, 2048, 12, 9), (63, 70000, 9, 3),           # short, many anchors: a wavefront each
    (9001, 32768, 30, 40), (9001, 32769, 30, 40), (40000, 32769, 200, 1 << 30),              # keys' tables of all anchors | of some
    (3000, 40000, 500, 1 << 30), (150000, 150000, 200, 1 << 30),                             # nearly too many keys | more than slots
    (3000, 98304, 9, 4), (3000, 98305, 9, 4),                                                # results told by the word | by the stream
    (16385, 5, 3, 2), (65537, 5, 3, 2), (262145, 5, 3, 2),                                   # turns of the first pass
])
def test_forms(P, ctx, n, k, tokens, stacks):                     # noqa: F811
    rng = np.random.default_rng([n, k, tokens])
    ref = sequence(rng, n, tokens, stacks)
    check(P, ctx, ref, perturbed(rng, ref), anchors(rng, n, k))
    check(P, ctx, ref, ref[:0], anchors(rng, n, k))
    check(P, ctx, perturbed(rng, ref), ref, anchors(rng, n, 7))


@pytest.mark.parametrize("n,k,tokens,stacks", [
    (1535, 12000, 1, 1), (1536, 12000, 2, 1), (1537, 12000, 30, 60),       # whole chunks of 512, one key and many
    (8191, 2100, 3, 2), (8192, 2100, 33, 1), (8193, 4000, 9, 30),           # two passes or one over the sequences, keys' bits
    (33000, 600, 25, 4), (131073, 300, 9, 1), (270000, 300, 9, 1),          # more than 64 chunks, chunks of 1,024 and 2,048
])
def test_numbered_chunks(P, ctx, n, k, tokens, stacks):           # noqa: F811
    rng = np.random.default_rng([n, k, tokens, 1])
    ref = sequence(rng, n, tokens, stacks)
    cur = perturbed(rng, ref)
    cur = np.concatenate([cur, ref[:n - len(cur)]])                 # of the same length
    check(P, ctx, ref, cur, anchors(rng, n, k))
    check(P, ctx, ref, cur[:n // 3], anchors(rng, n, k))


@pytest.mark.parametrize("m", [0, 1])
def test_the_most_anchors_over_the_fewest_operators(P, ctx, m):   # noqa: F811
    """2^24 anchors on one operator: the lowest keeps its counterpart, if there is one, and no launch is too large"""
    ref = sequence(np.random.default_rng(1), 1, 1, 1)
    ref["op_token"], ref["n_out"] = 1, 1
    cur = ref[:m].copy()
    cur["stack_hash"] += 1
    anc = np.zeros(1 << 24, dtype=W.ANCHOR_DT)
    r = P.ss_match_sequence(ctx, ref, cur, anc)
    assert (r["n_unmatched"], r["new_idx"][0], r["level"][0]) == (len(anc) - m, m - 1, 1 if m else 255)
    assert np.all(r["new_idx"][1:] == -1) and np.all(r["level"][1:] == 255)


@pytest.mark.parametrize("n,tokens", [(300, 7), (5000, 1500), (70000, 40), (20000, (1 << 18) - 1)])
def test_histograms(P, ctx, n, tokens):                           # noqa: F811
    rng = np.random.default_rng([n, tokens])
    ref = sequence(rng, n, tokens, 3)
    cur, anc = perturbed(rng, ref), anchors(rng, n, 40)
    r = P.ss_match_sequence(ctx, ref, cur, anc, flags=P.SS_MATCH_HISTOGRAM)
    assert (r["similar"], r["dot"], r["na"], r["nb"]) == oracle.similarity(cur["op_token"], ref["op_token"], histogram=True)
    assert np.array_equal(r["new_idx"], landings(ref, cur, anc)[0])
    for where in (cur, ref):
        bad = where.copy()
        bad["op_token"][len(bad) // 2] = 1 << 18
        for flags in (0, P.SS_MATCH_HISTOGRAM):
            with pytest.raises(P.SsError) as e:
                P.ss_match_sequence(ctx, bad if where is ref else ref, bad if where is cur else cur, anc, flags=flags)
            assert e.value.code == P.SS_E_INVAL
