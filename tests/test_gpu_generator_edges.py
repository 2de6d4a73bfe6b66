"""GPU parity of the policy generator where its list of operators over the limit changes form: lengths around the words of its
bit map and of the map over them, more entries than tensors, rounds that commit several, few or (accepting latency) one."""
import numpy as np
import pytest

import workloads as W
from test_gpu_generator import P, check_against_oracle, make_ctx, ops_with_phases      # noqa: F401  (fixture)
from test_oracle_generator import table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries,tensors", [(1, 6), (63, 40), (64, 40), (65, 40), (128, 12), (129, 60), (300, 20), (4200, 9)])
@pytest.mark.parametrize("bpo", [1 << 30, 3000, 120])
def test_entries_around_words(P, entries, tensors, bpo):           # noqa: F811
    rng = np.random.default_rng([entries, tensors, bpo])
    ramp = 24
    n = entries + 2 * ramp
    half = n // 2
    phases = [0] * half + [1] * (n - half)
    rows = []
    for _ in range(tensors):                                        # away from part of the plateau or from all of it
        lo, hi = (int(x) for x in np.sort(rng.integers(0, n - 2, 2)))
        if rng.random() < 0.6:
            lo, hi = int(rng.integers(0, ramp - 4)), int(rng.integers(n - ramp + 2, n - 2))
        if rng.random() < 0.2:
            hi = min(n - 2, lo + int(rng.integers(1, 8)))
        rows.append((lo, lo, max(hi, lo + 1), min(n - 1, max(hi, lo + 1) + 1), int(rng.integers(1, 9)) * 250))
    total = sum(r[4] for r in rows)
    rows.append((ramp, ramp, W.NONE_OP, n - ramp - 1, total))         # what makes the plateau; it has no backward use
    tab = table(rows)
    ev = W.transformer.events_of(tab)
    c = make_ctx(P, staging_bytes=4096, link_bytes_per_op=bpo)
    found = 0
    try:
        for share, layers, num in ((0.95, n // 6, 1), (0.6, n // 8, 4), (0.3, 3, 0)):
            limit = total + int(total * share * 0.5)
            found += check_against_oracle(P, c, ops_with_phases(phases), phases, tab, ev, n, limit, bpo, layers, layers,
                                          c_num=num, min_bytes=300) is not None
    finally:
        P.ss_destroy(c)
    assert found or entries == 1
