"""Box tests of the pattern search in tens of thousands of dimensions: what the distance's sum, taken in order, rounds
away must not let a box be passed over."""
import numpy as np
import pytest

import oracle as O
import paper_1706_02205_amd as K


# Points at the integers of one axis, those from 0 on off by eps in all other coordinates.  From -1 to 0 the distance is
# exactly 1, since eps^2 < 2^-53 is lost at each addition; four partial sums keep three quarters of it: 1 + 2e-12 and more.
@pytest.mark.parametrize("n,d", [(64, 24000), (100, 40000), (64, 7)])
def test_sums_that_lose_their_small_terms(n, d):
    x = np.zeros((n, d))
    x[:, 0] = np.arange(n) - n // 2
    x[n // 2:, 1:] = np.sqrt(0.99 * 2.0**-53)
    order = O.maximin(x)
    for rule in ("max", "min"):
        P = O.pattern(x, 1.0, O.RULE_MIN if rule == "min" else O.RULE_MAX, order)
        for threads in (1, 3):
            perm, l, colptr, rowidx = K.analyze(x, 1.0, rule, nthreads=threads).export()
            assert np.array_equal(perm, P.perm) and np.array_equal(l, P.l)
            assert np.array_equal(colptr, P.colptr) and np.array_equal(rowidx, P.rowidx)
