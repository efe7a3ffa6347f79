"""Small levels by teams of wavefronts: L, pivots and update counts equal the oracle's, whatever the row lengths."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1706_02205_amd as K
    return K


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# rows of at most 15, 16, 17, ... parents (chunks of 16), columns ending inside and at a 64-entry unit, indices at the
# ends of 32-bit words, long rows, and the pivot rules
@pytest.mark.parametrize("n,d,rho,policy", [(1, 2, 3.0, "zero"), (16, 2, 50.0, "zero"), (17, 2, 50.0, "zero"),
                                            (18, 2, 50.0, "shift"), (33, 1, 50.0, "zero"), (64, 2, 50.0, "zero"),
                                            (65, 2, 50.0, "zero"), (66, 3, 50.0, "shift"), (129, 2, 50.0, "zero"),
                                            (400, 2, 50.0, "shift"), (1500, 2, 2.0, "zero"), (6000, 3, 2.0, "zero")])
def test_team_levels_against_oracle_and_lane_walk(K, n, d, rho, policy):
    import oracle as O
    from paper_1706_02205_amd import workloads as W
    x = W.uniform_points(n, d, 900 + n)
    nu, ell = 0.5, 0.3
    tau = 1e-6 if policy == "shift" else 0.0
    P = O.pattern(x, rho)
    R = O.ichol(P, O.theta_on_pattern(P, nu, ell), O.PIVOT_SHIFT if policy == "shift" else O.PIVOT_ZERO, tau)
    plan = K.analyze(x, rho)
    print(f"[gpu] team n={n} d={d} rho={rho} max_row={plan.info()['max_row']}", flush=True)
    f = K.Factor(plan, "fp64")
    f.factorize(dev(x), nu, ell, policy, tau, count_updates=True)
    st = f.stats()
    assert np.array_equal(f.export_L(), R.L)
    assert (st.updates, st.nonpositive, st.shifted) == (R.updates, R.nonpositive, R.shifted)
    # mixed: the same updates in the same order as one lane per entry (all levels in one persistent launch)
    m = K.Factor(plan, "mixed")
    m.factorize(dev(x), nu, ell, "shift", 1e-6, count_updates=True)
    Lm, sm = m.export_L(), m.stats()
    m.set_schedule(1, 2**63 - 1)
    m.factorize(dev(x), nu, ell, "shift", 1e-6, count_updates=True)
    assert np.array_equal(Lm, m.export_L()) and sm == m.stats()


# the lane-per-entry kernel (here in persistent launches) with escaped row indices, small levels or not
@pytest.mark.parametrize("limit", [1, 3, 40])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_index_gap_escapes_in_the_lane_walk(K, limit, prec):
    from paper_1706_02205_amd import workloads as W
    x = W.uniform_points(3000, 2, 77)
    pol = ("zero", 0.0) if prec == "fp64" else ("shift", 1e-6)
    plan = K.analyze(x, 3.0)
    f = K.Factor(plan, prec)
    f.factorize(dev(x), 0.5, 0.2, *pol)
    want = f.export_L()
    plan.set_delta_limit(limit)
    g = K.Factor(plan, prec)
    g.set_schedule(1, 2**63 - 1)
    g.factorize(dev(x), 0.5, 0.2, *pol)
    assert np.array_equal(g.export_L(), want)
