"""The dense product in each of its workgroup shapes, on both sides of the sizes where they change."""
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


# 16 rows x 16 wavefronts, 32 x 4, 128 x 1; every register count of coordinates, padded (d = 4, 7, 19, 31) and full.
# Bound: a few ulp a kernel value and n additions in four-wide quads and at most 16 partial sums, of sum |Theta||X|.
@pytest.mark.parametrize("n,d,nu,nrhs", [(1, 8, 0.5, 1), (15, 4, 1.5, 3), (17, 7, 2.5, 9), (65, 31, 0.5, 4), (1023, 19, 1.5, 5),
                                         (6000, 20, 0.5, 8), (6001, 20, 2.5, 4), (28000, 3, 0.5, 1), (28001, 3, 1.5, 8),
                                         (30001, 32, 0.5, 2), (150001, 2, 0.5, 3), (150000, 1, 2.5, 5)])
def test_dense_shapes(K, n, d, nu, nrhs):
    import torch
    print(f"[gpu] dense n={n} d={d} nu={nu} nrhs={nrhs}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x = torch.rand(n, d, dtype=torch.float64, device="cuda", generator=g)
    X = torch.randn(n, nrhs, dtype=torch.float64, device="cuda", generator=g)
    ell = 0.2 * d**0.5
    Y = K.dense_matvec(x, X, nu, ell)
    rows = torch.unique(torch.cat([torch.arange(max(0, n - 20), n, device="cuda"),
                                   torch.randint(0, n, (40,), device="cuda", generator=g)]))
    s = torch.zeros(len(rows), n, dtype=torch.float64, device="cuda")
    for t in range(d):
        s += (x[rows, t, None] - x[None, :, t]) ** 2
    a = (2 * nu) ** 0.5 * s.sqrt() / ell
    th = torch.exp(-a) * {0.5: torch.ones_like(a), 1.5: 1 + a, 2.5: 1 + a + a * a / 3}[nu]
    err = (Y[rows] - th @ X).abs()
    assert bool((err <= 1e-12 * (th @ X.abs())).all())
    assert torch.equal(K.dense_matvec(x, X, nu, ell), Y)
