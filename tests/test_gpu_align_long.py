"""GPU parity of the sequence aligner where its kernels change form: one strip of 2,048 columns or several of 1,984, blocks of 32 steps, rows
walked on the host or on the GPU, mask tables in LDS or in device memory, paths that leave the tabulated window.
The whole pairing is compared exactly with the recurrence in Python integers, which is itself checked against the
oracle's textbook dynamic programme."""
import ctypes

import numpy as np
import pytest

from oracle.align import align_anchors
from helpers import ops_tuples
from test_gpu_align import ops_arr, P, ctx          # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def pairing(ref, cur):
    """canonical alignment: read from the end, equal operators pair, else left if that loses nothing, else up"""
    n, m = len(ref), len(cur)
    full = (1 << m) - 1
    at = {}
    for j, k in enumerate(cur):
        at.setdefault(k, bytearray(m // 8 + 1))[j >> 3] |= 1 << (j & 7)
    mask = {k: int.from_bytes(b, "little") for k, b in at.items()}
    rows, v = [], full
    for k in ref:
        u = v & mask.get(k, 0)
        v = ((v + u) | (v - u)) & full
        rows.append(v.to_bytes(m // 8 + 1, "little"))
    pair = np.full(n, -1, dtype=np.int32)
    i, j = n, m
    while i and j:
        if ref[i - 1] == cur[j - 1]:
            i, j = i - 1, j - 1
            pair[i] = j
        elif rows[i - 1][(j - 1) >> 3] >> ((j - 1) & 7) & 1:
            j -= 1
        else:
            i -= 1
    return pair


def perturbed(rng, keys, foreign):
    keep = keys[rng.random(len(keys)) >= 0.1]
    k = max(1, len(keep) // 10)
    return np.insert(keep, rng.integers(0, len(keep) + 1, k), foreign + rng.integers(0, 5, k))


def test_the_reference_here_is_the_oracles(P):                    # noqa: F811
    rng = np.random.default_rng(1)
    for _ in range(20):
        n, m, a = rng.integers(1, 60), rng.integers(1, 60), rng.integers(1, 9)
        ref, cur = rng.integers(0, a, n), rng.integers(0, a, m)
        want = align_anchors(ops_tuples(ops_arr(ref)), ops_tuples(ops_arr(cur)), [])["ref_to_cur"]
        assert np.array_equal(pairing(ref.tolist(), cur.tolist()), want)


@pytest.mark.parametrize("n,m,alpha", [
    (1, 2048, 3), (31, 2049, 5), (33, 2047, 5), (64, 4096, 40), (97, 4097, 7), (400, 6145, 250),     # strip and block edges
    (30, 1984, 5), (65, 3968, 7), (96, 3969, 300), (1, 5953, 3),
    (8191, 4000, 30), (8193, 4097, 30), (16300, 1900, 12), (16500, 1900, 12),                         # host walk, GPU walk
    (9000, 9001, 254), (9000, 9001, 255), (9000, 9001, 256), (9000, 9001, 3000),                      # LDS masks, masks in memory
    (8704, 9000, 40), (8705, 9000, 40),                                                               # groups of blocks walked back
    (65536, 600, 200), (700, 40000, 60), (40000, 700, 60),                                            # ids beyond LDS, steep and flat
])
def test_random_and_perturbed_at_the_edges(P, ctx, n, m, alpha):  # noqa: F811
    rng = np.random.default_rng([n, m, alpha])
    ref = rng.integers(0, alpha, n)
    ref[:min(n, alpha)] = np.arange(min(n, alpha))               # every key is there
    for cur in (rng.integers(0, alpha, m), perturbed(rng, ref, alpha)[:m]):
        lib = P.ss_align_sequence(ctx, ops_arr(ref), ops_arr(cur))
        assert np.array_equal(lib["ref_to_cur"], pairing(ref.tolist(), cur.tolist())), (n, m, alpha)
        assert lib["lcs"] == int((lib["ref_to_cur"] >= 0).sum())


@pytest.mark.parametrize("n", [9000, 20000])
def test_long_gaps_leave_the_window(P, ctx, n):                   # noqa: F811
    """thousands of operators missing or foreign in one piece: the path runs along the edge of what is tabulated, off
    it, and back"""
    rng = np.random.default_rng(n)
    ref = np.tile(rng.integers(0, 30, 500), n // 500)
    for cur in (np.concatenate([ref[:n // 3], 30 + rng.integers(0, 3, 3000), ref[n // 3:]]),
                np.concatenate([ref[:n // 4], ref[n // 2:]]),
                np.concatenate([30 + rng.integers(0, 3, 400), ref[n // 3:], 30 + rng.integers(0, 3, 5000)])):
        lib = P.ss_align_sequence(ctx, ops_arr(ref), ops_arr(cur))
        assert np.array_equal(lib["ref_to_cur"], pairing(ref.tolist(), cur.tolist()))


@pytest.mark.parametrize("n,m,alpha", [
    (500, 6145, 250), (700, 40000, 60), (9000, 9001, 254), (9000, 9001, 3000),       # walked on the host, on the GPU, wide ids
    (1154, 1156, 40),                                                                # one strip: nothing to wait for
])
def test_strips_that_give_up_waiting_are_started_one_by_one(P, ctx, n, m, alpha):    # noqa: F811
    """a limit of zero: a strip that finds its neighbour's first word missing leaves at once, the kernel ends, and the call
    still gives the pairing; so does the next one under the usual limit"""
    lib = ctypes.CDLL(P.LIB_PATH)
    lib.ss_align_wait_limit.argtypes, lib.ss_align_wait_limit.restype = [ctypes.c_void_p, ctypes.c_uint32], ctypes.c_uint32
    rng = np.random.default_rng([n, m, alpha, 1])
    ref = rng.integers(0, alpha, n)
    ref[:min(n, alpha)] = np.arange(min(n, alpha))
    cur = rng.integers(0, alpha, m)
    want = pairing(ref.tolist(), cur.tolist())
    x, y = ops_arr(ref), ops_arr(cur)
    anc = np.zeros(50, dtype=P.ANCHOR_DT)
    anc["ref_op"] = rng.integers(0, n, 50)
    usual, many = 1 << 20, m > 2048
    before = lib.ss_align_wait_limit(ctx, 0)
    try:
        assert np.array_equal(P.ss_align_sequence(ctx, x, y)["ref_to_cur"], want)
        got = P.ss_match_sequence(ctx, x, y, anc, flags=P.SS_MATCH_ALIGN)
    finally:
        after = lib.ss_align_wait_limit(ctx, usual)
    assert after - before == (2 if many else 0)
    again = P.ss_match_sequence(ctx, x, y, anc, flags=P.SS_MATCH_ALIGN)
    assert np.array_equal(got["new_idx"], again["new_idx"]) and np.array_equal(got["level"], again["level"])
    assert np.array_equal(P.ss_align_sequence(ctx, x, y)["ref_to_cur"], want)
    assert lib.ss_align_wait_limit(ctx, usual) == after


@pytest.mark.parametrize("n,m,alpha", [
    (1, 1, 1), (4095, 1, 3), (4064, 32, 4), (1, 33, 2), (31, 64, 5), (2048, 2048, 40), (2047, 2049, 40), (2049, 2048, 40),
    (2080, 2016, 30), (2048, 2017, 30), (1000, 1100, 254), (1000, 1100, 255), (1000, 1100, 256), (1500, 2000, 1500),
])
def test_short_sequences_in_one_workgroup(P, n, m, alpha):           # noqa: F811
    """one strip and both sequences' keys in one workgroup, or just not; lanes with and without a word; ids of 16 and of 32
    bits, also where a new context's scratch turns out too small for the masks"""
    rng = np.random.default_rng([n, m, alpha, 2])
    ref, cur = rng.integers(0, alpha, n), rng.integers(0, alpha, m)
    cur[:min(m, alpha)] = np.arange(min(m, alpha))                   # every key is there
    want = pairing(ref.tolist(), cur.tolist())
    c = P.ss_create(P.ss_config_default())
    for _ in range(3):
        lib = P.ss_align_sequence(c, ops_arr(ref), ops_arr(cur))
        assert np.array_equal(lib["ref_to_cur"], want)
        assert lib["n_keys"] == min(m, alpha)
    P.ss_destroy(c)
