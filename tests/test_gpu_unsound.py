"""Summed backward columns and factors with shifted pivots: such a factor keeps the sequential order, instance by instance."""
import numpy as np
import pytest

import oracle as O
from paper_1706_02205_amd import workloads as W

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


# Three instances in every order, the one with lengthscale 5 shifting some 300 pivots, the other two none (their least
# pivot is five times tau): each is solved bitwise as alone, by kc_solve, by the fused call and by a captured graph.
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("order", [(0, 1, 2), (2, 0, 1)])
def test_instance_of_a_batch_with_shifted_pivots_elsewhere(K, prec, order):
    nu, rho, tau = 0.5, 4.0, 1e-3
    pts = [W.uniform_points(5000, 2, 4311), W.uniform_points(1200, 2, 4312), W.uniform_points(4000, 2, 4313)]
    lens = np.array([0.05, 0.3, 5.0])
    xs, ells = [pts[i] for i in order], lens[list(order)]
    print(f"[gpu] batch of sound and unsound instances {prec} {order}", flush=True)
    b = [W.gaussian_rhs(len(x), 3, 4500 + i) for i, x in enumerate(xs)]
    plan = K.analyze_batched(xs, rho)
    xd, ed, bd = dev(np.concatenate(xs)), dev(ells), dev(np.concatenate(b))
    f = K.Factor(plan, prec)
    f.factorize_batched(xd, nu, ed, "shift", tau)
    got = f.solve(bd).cpu().numpy()
    assert np.array_equal(f.factorize_solve(xd, bd, nu, pivot="shift", tau=tau, ell_dev=ed).cpu().numpy(), got)
    g = f.capture(xd, bd, nu, ell_dev=ed, pivot="shift", tau=tau)
    for _ in range(3):
        out = g.launch()
        f.solve(bd)
        assert np.array_equal(out.cpu().numpy(), got)
    o0 = 0
    for i, (x, ell) in enumerate(zip(xs, ells)):
        alone_plan = K.analyze(x, rho)
        alone = K.Factor(alone_plan, prec)
        alone.factorize(dev(x), nu, float(ell), "shift", tau)
        assert (alone.stats().shifted > 0) == (ell == 5.0)
        want = alone.solve(dev(b[i])).cpu().numpy()
        if len(x) > 2049:  # with columns past the top block that a sound factor sums
            cols = np.diff(alone_plan.export()[2]) - 1
            assert ((cols > 256) & (np.arange(len(x)) > np.nonzero(cols > 2048)[0].max())).any()
        assert np.array_equal(got[o0:o0 + len(x)], want), f"instance {i}"
        o0 += len(x)


# Notes beyond the 64 values that one workgroup clears: the long instance last of 2, 33 and 70, unsound and sound again.
@pytest.mark.parametrize("count", [2, 33, 70])
def test_notes_of_many_instances_are_cleared(K, count):
    nu, rho, x = 0.5, 4.0, W.uniform_points(5000, 2, 4311)
    print(f"[gpu] notes of {count} instances", flush=True)
    xs = [W.uniform_points(3 + i % 5, 2, i) for i in range(count - 1)] + [x]
    b = W.gaussian_rhs(sum(map(len, xs)), 2, 4600)
    xd, ed, bd = dev(np.concatenate(xs)), dev(np.full(count, 0.05)), dev(b)
    f = K.Factor(K.analyze_batched(xs, rho), "fp64")
    f.factorize_batched(xd, nu, ed, "shift", 1e-3)
    assert f.stats().shifted == 0
    want = f.solve(bd).cpu().numpy()
    alone = K.Factor(K.analyze(x, rho), "fp64")
    alone.factorize(dev(x), nu, 0.05, "shift", 1e-3)
    assert np.array_equal(want[-len(x):], alone.solve(dev(b[-len(x):])).cpu().numpy())
    f.factorize_batched(xd, nu, ed, "shift", 0.5)
    assert f.stats().shifted > 0
    alone.factorize(dev(x), nu, 0.05, "shift", 0.5)
    got = f.solve(bd).cpu().numpy()
    assert np.array_equal(got[-len(x):], alone.solve(dev(b[-len(x):])).cpu().numpy())
    f.factorize_batched(xd, nu, ed, "shift", 1e-3)
    assert np.array_equal(f.solve(bd).cpu().numpy(), want)


# Positions past the last long column see no summed piece but these columns, so there the sequential order shows bit for
# bit: finite after shifted pivots; overflowing, with the oracle's infinities and NaN at their places; and not so for a
# sound factor, which sums.
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,d,rho,nu,ell,tau,kind", [(6000, 2, 6.0, 0.5, 0.3, 0.5, "shifted"),
                                                     (4000, 3, 3.0, 2.5, 0.2, 1e-9, "overflowing"),
                                                     (6000, 2, 6.0, 0.5, 0.3, 1e-9, "sound")])
def test_order_past_the_top_block(K, prec, n, d, rho, nu, ell, tau, kind):
    print(f"[gpu] order past the top block: {kind} {prec}", flush=True)
    x = W.uniform_points(n, d, 31)
    plan = K.analyze(x, rho)
    perm, _, colptr, _ = plan.export()
    cols = np.diff(colptr) - 1
    top = int(np.nonzero(cols > 2048)[0].max()) + 1
    assert ((cols > 256) & (np.arange(n) >= top)).any()
    assert np.bincount(plan.levels()).max() < 1024  # no forward level is summed
    b = W.gaussian_rhs(n, 2, 32)
    f = K.Factor(plan, prec)
    f.factorize(dev(x), nu, ell, "shift", tau)
    st = f.stats()
    ref = O.solve(O.pattern(x, rho), f.export_L(), b)[perm[top:]]
    got = f.solve(dev(b)).cpu().numpy()[perm[top:]]
    if kind == "sound":
        assert st.shifted == 0 and st.nonfinite == 0
        assert not np.array_equal(got, ref) and np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
        return
    assert st.shifted > 0
    assert np.array_equal(got, ref, equal_nan=True)
    if kind == "overflowing":
        assert np.isnan(ref).any() and np.isinf(ref).any()
        if prec == "fp64":
            assert np.isfinite(ref).any()
    else:
        assert np.isfinite(ref).all()
