"""The pattern by one thread (rows put in order by transposition) and by several (sorted columns): the oracle's, with
blocks of a leaf's points on both sides of 32 (coinciding points share one leaf)."""
import numpy as np
import pytest

import oracle as O
import paper_1706_02205_amd as K
from paper_1706_02205_amd import workloads as W


def points(kind):
    if kind == "uniform2d":
        return W.uniform_points(3000, 2, 5)
    if kind == "uniform3d":
        return W.uniform_points(2000, 3, 6)
    if kind == "sphere20":
        return W.embedded_sincos(1500, 7)
    if kind == "five":
        return W.uniform_points(900, 5, 8)
    if kind == "duplicates":
        return np.ascontiguousarray(np.repeat(W.uniform_points(40, 2, 9), [1, 33, 70, 2] * 10, axis=0))
    return np.zeros((70, 3))


@pytest.mark.parametrize("kind", ["uniform2d", "uniform3d", "sphere20", "five", "duplicates", "one place"])
@pytest.mark.parametrize("rule", ["max", "min"])
def test_pattern_by_one_and_by_several_threads(kind, rule):
    x = points(kind)
    P = O.pattern(x, 2.5, O.RULE_MIN if rule == "min" else O.RULE_MAX)
    for threads in (1, 3):
        perm, l, colptr, rowidx = K.analyze(x, 2.5, rule, nthreads=threads).export()
        assert np.array_equal(perm, P.perm) and np.array_equal(l, P.l)
        assert np.array_equal(colptr, P.colptr) and np.array_equal(rowidx, P.rowidx)
