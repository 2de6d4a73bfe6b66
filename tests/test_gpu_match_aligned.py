"""GPU parity of aligned matching (SS_MATCH_ALIGN), whose cosine is taken by the aligner's first kernel: sums, verdict and landings at the
lengths where one workgroup or many read the operators, with one sequence longer, few keys and many, and tokens out of range."""
import numpy as np
import pytest

from test_gpu_align import P, ctx                                  # noqa: F401  (fixtures)
from test_gpu_align_long import pairing

pytestmark = pytest.mark.gpu


def operators(P, keys):                                            # noqa: F811
    ops = np.zeros(len(keys), dtype=P.OP_DT)
    ops["op_token"] = 1 + keys * 37 % 5000
    ops["stack_hash"] = 5 + keys // 5000
    ops["sig"] = 0x0101
    ops["n_out"] = 1 + keys % 2
    return ops


@pytest.mark.parametrize("n,m,keys", [(1, 1, 1), (1, 5, 2), (64, 63, 5), (1024, 1025, 30), (2047, 2049, 40), (4095, 1, 3), (1, 4095, 3),
                                      (2048, 2049, 40), (2500, 1700, 300), (5000, 4900, 30), (700, 9000, 20), (70000 // 8, 9000, 2000)])
def test_sums_and_landings(P, ctx, n, m, keys):                    # noqa: F811
    rng = np.random.default_rng([n, m, keys])
    rk, ck = rng.integers(0, keys, n), rng.integers(0, keys, m)
    if n == m:
        ck[0] += 1                                                 # the same sequence twice is another path
    ref, cur = operators(P, rk), operators(P, ck)
    anc = np.zeros(40, dtype=P.ANCHOR_DT)
    anc["ref_op"] = rng.integers(0, n + 2, 40)
    anc["out_slot"] = rng.integers(0, 3, 40)
    pair = pairing(rk.tolist(), ck.tolist())
    a, b = np.zeros(max(n, m), dtype=np.int64), np.zeros(max(n, m), dtype=np.int64)
    a[:m], b[:n] = cur["op_token"], ref["op_token"]
    dot, na, nb = int((a * b).sum()), int((a * a).sum()), int((b * b).sum())
    for _ in range(2):
        got = P.ss_match_sequence(ctx, ref, cur, anc, flags=P.SS_MATCH_ALIGN)
        assert (got["dot"], got["na"], got["nb"]) == (dot, na, nb)
        assert got["similar"] == (20 * abs(n - m) < n and dot > 0 and 400 * dot * dot > 361 * na * nb)
        want = [int(pair[i]) if i < n and pair[i] >= 0 and s < cur["n_out"][pair[i]] else -1 for i, s in anc.tolist()]
        assert got["new_idx"].tolist() == want
        assert got["level"].tolist() == [3 if j >= 0 else 255 for j in want]
        assert got["n_unmatched"] == want.count(-1)


@pytest.mark.parametrize("n,m", [(100, 90), (3000, 2900)])
@pytest.mark.parametrize("where", ["ref", "cur"])
def test_tokens_out_of_range(P, ctx, n, m, where):                 # noqa: F811
    rng = np.random.default_rng(n)
    ref, cur = operators(P, rng.integers(0, 20, n)), operators(P, rng.integers(0, 20, m))
    anc = np.zeros(3, dtype=P.ANCHOR_DT)
    seq = ref if where == "ref" else cur
    seq["op_token"][-1] = (1 << 18) - 1
    P.ss_match_sequence(ctx, ref, cur, anc, flags=P.SS_MATCH_ALIGN)
    seq["op_token"][-1] = 1 << 18
    with pytest.raises(P.SsError) as e:
        P.ss_match_sequence(ctx, ref, cur, anc, flags=P.SS_MATCH_ALIGN)
    assert e.value.code == P.SS_E_INVAL
