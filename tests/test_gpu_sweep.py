"""Small sweep levels by a workgroup per row: bitwise the sequential substitution at every block length and width."""
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


# full patterns, so that rows and columns take every length up to n - 1: below, at and above a step of 16 entries and a
# block of 256 (and of 320, the width when a sweep level shares the factorization's launch), several blocks, 2049 = the
# longest column summed in sequence
@pytest.mark.parametrize("n,nrhs", [(2, 1), (17, 2), (18, 9), (257, 1), (258, 5), (321, 3), (322, 8), (530, 7), (700, 16),
                                    (2049, 4)])
def test_every_row_length_bitwise(K, n, nrhs):
    import torch
    import oracle as O
    from paper_1706_02205_amd import workloads as W
    x = W.uniform_points(n, 2, 400 + n)
    rho = 1e6
    P = O.pattern(x, rho)
    assert P.nnz == n * (n + 1) // 2
    R = O.ichol(P, O.theta_on_pattern(P, 0.5, 0.3))
    b = W.gaussian_rhs(n, nrhs, n)
    ref = O.solve(P, R.L, b)
    print(f"[gpu] sweep n={n} nrhs={nrhs}", flush=True)
    f = K.Factor(K.analyze(x, rho), "fp64")
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()
    f.factorize(xd, 0.5, 0.3)
    assert np.array_equal(f.solve(bd).cpu().numpy(), ref)
    assert np.array_equal(f.factorize_solve(xd, bd, 0.5, 0.3).cpu().numpy(), ref)
    g = f.capture(xd, bd, 0.5, 0.3)
    for _ in range(3):
        out = g.launch()
        f.solve(bd)
        assert np.array_equal(out.cpu().numpy(), ref)


# A plan with columns of more than 2,048 entries: later columns of more than 256 are summed across a workgroup, within
# 1e-12 of the largest component; after shifted pivots (here nearly all) every column at or above the top block keeps the
# sequential order, so that overflow leaves the same infinities and NaN as a level-by-level solve of the same factor.
@pytest.mark.parametrize("prec,nrhs", [("fp64", 1), ("fp64", 9), ("mixed", 4)])
def test_summed_columns(K, prec, nrhs):
    import torch
    import oracle as O
    from paper_1706_02205_amd import workloads as W
    n = 6000
    x = W.uniform_points(n, 2, 31)
    plan = K.analyze(x, 6.0)
    _, _, colptr, _ = plan.export()
    cols = np.diff(colptr) - 1
    top = int(np.nonzero(cols > 2048)[0].max()) + 1
    assert ((cols > 256) & (np.arange(n) >= top)).any()
    xd = torch.from_numpy(x).cuda()
    b = W.gaussian_rhs(n, nrhs, 32)
    bd = torch.from_numpy(b).cuda()
    f = K.Factor(plan, prec)
    f.factorize(xd, 0.5, 0.3)
    P = O.pattern(x, 6.0)
    ref = O.solve(P, f.export_L(), b)
    got = f.solve(bd).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    assert np.array_equal(f.factorize_solve(xd, bd, 0.5, 0.3).cpu().numpy(), got)
    # the note of unsound factors: shifted pivots, then a sound factorization again
    f.factorize(xd, 0.5, 0.3, "shift", 0.5)
    assert f.stats().shifted > 0
    a = f.solve(bd).cpu().numpy()
    ref = O.solve(P, f.export_L(), b)
    fine = np.isfinite(ref).all()
    assert not fine or np.abs(a - ref).max() <= 1e-12 * np.abs(ref).max()
    f.theta(xd, 0.5, 0.3)
    assert np.array_equal(f.solve(bd).cpu().numpy(), a, equal_nan=True)
    assert np.array_equal(f.factorize_solve(xd, bd, 0.5, 0.3).cpu().numpy(), got)
