"""GPU parity of the walk back over long sequences where its tables change: rows without a column to stop in."""
import numpy as np
import pytest

from helpers import ops_tuples                                     # noqa: F401
from test_gpu_align import ops_arr, P, ctx                         # noqa: F401  (fixtures)
from test_gpu_align_long import pairing, perturbed

pytestmark = pytest.mark.gpu


def same(P, ctx, ref, cur):
    lib = P.ss_align_sequence(ctx, ops_arr(ref), ops_arr(cur))
    assert np.array_equal(lib["ref_to_cur"], pairing(ref.tolist(), cur.tolist()))


def test_stretches_that_have_nothing_in_common(P, ctx):            # noqa: F811
    """rows in which no column of a tile is equal or steps up, and a current sequence that ends or begins with them"""
    rng = np.random.default_rng(7)
    ref = rng.integers(0, 30, 10000)
    other = 50 + rng.integers(0, 30, 10000)
    for cur in (np.concatenate([other[:4000], ref[4000:]]), np.concatenate([ref[:6000], other[6000:]]),
                np.concatenate([ref[:3000], other[3000:7000], ref[7000:]]), other, np.where(np.arange(10000) // 700 % 2, ref, other)):
        same(P, ctx, ref, cur)
