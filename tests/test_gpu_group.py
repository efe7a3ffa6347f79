"""Supernodal groups: parents taken 256 and 128 at a time, units per level on both sides of that rule."""
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


# FP32 updates of |P| parents are off by at most |P| 2^-24 of sum |L_ki L_gi| <= 1 (rows of L have norm <= 1), divided by
# the pivot's root: entries agree with the entry-wise mixed factor within 2 |P| 2^-24 / min pivot, carried on by later
# columns (a factor of 10 for those).
@pytest.mark.parametrize("n,d,rho", [(1, 3, 3.0), (17, 3, 50.0), (300, 3, 50.0), (1200, 2, 3.0), (3000, 3, 3.0),
                                     (12000, 3, 2.0)])
def test_groups_against_entrywise(K, n, d, rho):
    import torch
    from paper_1706_02205_amd import workloads as W
    x = W.uniform_points(n, d, 70 + n)
    plan = K.analyze_supernodal(x, rho)
    xd = torch.from_numpy(x).cuda()
    print(f"[gpu] groups n={n} d={d} rho={rho} max_row={plan.info()['max_row']}", flush=True)
    f = K.Factor(plan, "mixed")
    f.factorize(xd, 0.5, 0.2, "shift", 1e-6)
    Lg, sg = f.export_L(), f.stats()
    f.factorize(xd, 0.5, 0.2, "shift", 1e-6)
    assert np.array_equal(f.export_L(), Lg)
    f.use_groups(False)
    f.factorize(xd, 0.5, 0.2, "shift", 1e-6)
    Le, se = f.export_L(), f.stats()
    assert sg.shifted == se.shifted == 0 and sg.nonfinite == 0
    _, _, colptr, _ = plan.export()
    bound = 20 * plan.info()["max_row"] * 2.0**-24 / Le[colptr[:-1]].min()
    assert np.abs(Lg - Le).max() <= bound
