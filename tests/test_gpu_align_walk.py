"""GPU parity of the walk back over long sequences where its windows, blocks and tables change: paths that stay inside the narrow
windows, leave them on either side or only just, lengths about the limit for trying them, remainders of blocks and groups, rows
without a column to stop in, 16-bit and wide ids."""
import numpy as np
import pytest

from helpers import ops_tuples                                     # noqa: F401
from test_gpu_align import ops_arr, P, ctx                         # noqa: F401  (fixtures)
from test_gpu_align_long import pairing, perturbed

pytestmark = pytest.mark.gpu


def same(P, ctx, ref, cur):
    lib = P.ss_align_sequence(ctx, ops_arr(ref), ops_arr(cur))
    assert np.array_equal(lib["ref_to_cur"], pairing(ref.tolist(), cur.tolist()))


@pytest.mark.parametrize("keys", [40, 900])
@pytest.mark.parametrize("shift", [120, 383, 384, 400, 511, 512, 640, 641, 900, 1024, 1300])
def test_paths_beside_the_diagonal(P, ctx, keys, shift):           # noqa: F811
    """a piece of foreign operators before the middle and as many missing after it, and the other way round"""
    rng = np.random.default_rng([keys, shift])
    n = 9100
    ref = perturbed(rng, np.tile(rng.integers(0, keys, 700), 14)[:n], keys)
    n = len(ref)
    a, b = n // 5, 4 * n // 5
    foreign = keys + 5 + rng.integers(0, 4, shift)
    same(P, ctx, ref, perturbed(rng, np.concatenate([ref[:a], foreign, ref[a:b], ref[b + shift:]]), keys))
    same(P, ctx, ref, np.concatenate([ref[:a], ref[a + shift:b], foreign, ref[b:]]))


@pytest.mark.parametrize("n", [8705, 8703, 9216, 9217, 16384, 16385])
@pytest.mark.parametrize("more", [-513, -512, 0, 1, 512, 513])
def test_lengths_about_the_limit_and_remainders(P, ctx, n, more):  # noqa: F811
    rng = np.random.default_rng([n, more + 1000])
    ref = rng.integers(0, 25, n)
    cur = np.concatenate([ref, 60 + rng.integers(0, 5, max(0, more))])[:n + min(0, more)]
    same(P, ctx, ref, cur)
    same(P, ctx, ref, perturbed(rng, ref, 25)[:n])


@pytest.mark.parametrize("n,m", [(3263, 3250), (3264, 3264), (3265, 3265), (3270, 3270), (6598, 2000), (6800, 1900),     # rows of 1,700 KiB
                                 (2000, 8000), (2000, 8001), (1500, 6001), (1300, 11000), (1400, 5600)])               # four times as long
def test_walked_on_the_host_or_on_the_gpu(P, ctx, n, m):           # noqa: F811
    rng = np.random.default_rng([n, m])
    base = rng.integers(0, 30, max(n, m))
    cut = [base[np.sort(rng.choice(len(base), k, replace=False))] for k in (n, m)]
    same(P, ctx, *cut)


def test_stretches_that_have_nothing_in_common(P, ctx):            # noqa: F811
    """rows in which no column of a tile is equal or steps up, and a current sequence that ends or begins with them"""
    rng = np.random.default_rng(7)
    ref = rng.integers(0, 30, 10000)
    other = 50 + rng.integers(0, 30, 10000)
    for cur in (np.concatenate([other[:4000], ref[4000:]]), np.concatenate([ref[:6000], other[6000:]]),
                np.concatenate([ref[:3000], other[3000:7000], ref[7000:]]), other, np.where(np.arange(10000) // 700 % 2, ref, other)):
        same(P, ctx, ref, cur)


@pytest.mark.parametrize("n,m", [(2600, 2700), (700, 4000), (9000, 9001)])
def test_few_keys_and_many_in_turn(P, n, m):                       # noqa: F811
    """rows are launched before the number of keys is known, unless the call before had many: 255 and 256 keys, each after either,
    the first ones on a new context whose scratch is small"""
    rng = np.random.default_rng([n, m, 3])
    c = P.ss_create(P.ss_config_default())
    try:
        for keys in (256, 255, 256, 1500, 40, 255, 900, 256, 30, 30):
            ref = rng.integers(0, keys, n)
            cur = perturbed(rng, np.tile(ref, 1 + m // n), keys - 5)[:m] if m > n and keys > 300 else rng.integers(0, keys, m)
            cur[:keys] = np.arange(keys)
            lib = P.ss_align_sequence(c, ops_arr(ref), ops_arr(cur))
            assert np.array_equal(lib["ref_to_cur"], pairing(ref.tolist(), cur.tolist())), keys
            assert lib["n_keys"] == len(set(cur.tolist()))
    finally:
        P.ss_destroy(c)


@pytest.mark.parametrize("period", [1, 2, 3, 4, 5, 7, 64])
def test_blocks_of_short_runs(P, ctx, period):                     # noqa: F811
    """a foreign operator in every `period`-th place: 64 to 0 ends of runs to a block, 32 and 48 rows to the first
    sixteen on either side of where it is gone through row by row; the others equal all along, or drawn anew"""
    rng = np.random.default_rng(period)
    ref = rng.integers(0, 20, 9300)
    cur = np.where(np.arange(len(ref)) % period == 0, 50, ref)
    same(P, ctx, ref, cur)
    same(P, ctx, ref, np.where(np.arange(len(ref)) // 640 % 2, rng.integers(0, 20, len(ref)), cur))


@pytest.mark.parametrize("keys", [40, 900])
@pytest.mark.parametrize("gap", [130, 192, 256, 300, 4032, 4096, 4170, 8400])
def test_far_to_the_left_in_one_row(P, ctx, keys, gap):            # noqa: F811
    """columns without a stop: some words of them, as many as are looked at together and more, at the end, between equal stretches
    and at the front of cur"""
    rng = np.random.default_rng([keys, gap])
    ref = rng.integers(0, keys, 9050)
    foreign = np.full(gap, keys + 7)
    for at in (len(ref), 5003, 4992, 64, 0):
        same(P, ctx, ref, np.concatenate([ref[:at], foreign, ref[at:]]))
    same(P, ctx, ref, np.concatenate([foreign, ref[200:300], foreign, ref[4000:4001], foreign]))


@pytest.mark.parametrize("keys", [40, 900])
@pytest.mark.parametrize("at", [2, 7, 8, 9, 15, 16, 17, 60, 135])
def test_walks_that_go_on_where_the_path_has_left_the_windows(P, ctx, keys, at):         # noqa: F811
    """the path leaves the narrow windows about block `at` from the end: within a group of eight blocks and at its first and last one,
    in the last blocks of the walk, to either side; it stays beside the diagonal, comes back or leaves the second windows too"""
    rng = np.random.default_rng([keys, at])
    n = 9100
    ref = rng.integers(0, keys, n)
    x = max(0, n - 64 * at)
    foreign = keys + 5 + rng.integers(0, 4, 3000)
    for shift in (650, 1700):
        same(P, ctx, ref, np.concatenate([foreign[:shift], ref[:max(0, x - shift)], ref[x:]]))
        same(P, ctx, ref, np.concatenate([ref[shift:x], foreign[:min(shift, x)], ref[x:]]))
        same(P, ctx, ref, np.concatenate([ref[:x // 2], foreign[:shift], ref[x // 2:max(x // 2, x - shift)], ref[x:]]))
    y = max(0, x - 2500)
    same(P, ctx, ref, np.concatenate([ref[:y // 2], foreign[:1600], ref[y // 2:max(y // 2, y - 800)], ref[y:max(y, x - 800)], ref[x:]]))


@pytest.mark.parametrize("n,m", [(3300, 3300), (4000, 4500), (4288, 4288), (4289, 4350), (4800, 4300), (8000, 3000), (2200, 4400), (2200, 4401),
                                 (5100, 8191), (5100, 8192), (12000, 2047), (12000, 2048), (20000, 900),
                                 (4000, 5024), (4000, 5025), (5025, 4000)])
def test_tables_of_all_columns(P, ctx, n, m):                      # noqa: F811
    """paths near the diagonal, far beside it and along the edges, where all columns are tabulated and where they just aren't"""
    rng = np.random.default_rng([n, m, 8])
    base = rng.integers(0, 35, max(n, m))
    ref, cur = base[:n], base[:m]
    same(P, ctx, ref, cur)
    same(P, ctx, base[-n:], base[-m:])
    same(P, ctx, ref, perturbed(rng, np.resize(ref, m), 35)[:m])
    k = min(n, m) // 2
    same(P, ctx, ref, np.concatenate([np.full(m - k, 70), ref[:k]]))
    same(P, ctx, ref, np.concatenate([ref[-k:], 70 + rng.integers(0, 3, m - k)]))
    same(P, ctx, ref, 100 + rng.integers(0, 30, m))
