"""The dense product of points far from the origin, in more than three dimensions: coordinates are subtracted before
anything is rounded, so a kernel value is as accurate as at the origin."""
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


# Unit vectors as right-hand sides, so that a result is one kernel value.  Bound, relative, u = 2^-53: the distance is off
# by (d / 2 + 3) u and the argument a <= 5 by two roundings more, which the kernel takes up a-fold, and the exponential
# with its polynomial by 8 u; doubled.  Sizes on both sides of the row splits, one register count each.
@pytest.mark.parametrize("offset", [0.0, 1e3, 1e6])
@pytest.mark.parametrize("n,d,nu", [(300, 4, 0.5), (301, 8, 1.5), (6001, 20, 0.5), (299, 31, 2.5), (28003, 6, 0.5),
                                    (30003, 21, 1.5)])
def test_offset_points(K, n, d, nu, offset):
    import torch
    print(f"[gpu] dense offset n={n} d={d} nu={nu} offset={offset:g}", flush=True)
    rng = np.random.default_rng(n + d)
    x = offset + rng.random((n, d))
    ell = 0.45 * d**0.5
    cols = rng.choice(n, 8, replace=False)
    X = np.zeros((n, 8))
    X[cols, np.arange(8)] = 1.0
    Y = K.dense_matvec(torch.from_numpy(x).cuda(), torch.from_numpy(X).cuda(), nu, ell).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(n, 300)), cols, np.arange(n - 10, n)]))
    xl = x.astype(np.longdouble)
    r = np.sqrt(((xl[rows, None] - xl[None, cols]) ** 2).sum(-1))
    a = np.sqrt(np.longdouble(2 * nu)) * r / np.longdouble(ell)
    assert a.max() <= 5
    th = np.exp(-a) * {0.5: 1, 1.5: 1 + a, 2.5: 1 + a + a * a / 3}[nu]
    err = np.abs(Y[rows] - th) / th
    print(f"[gpu] largest relative error {float(err.max()):.2e}", flush=True)
    assert err.max() <= 2 * (5 * (d / 2 + 5) + 8) * 2.0**-53
