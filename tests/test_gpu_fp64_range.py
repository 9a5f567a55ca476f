"""FP64 divisions at the ends of the range, against the oracle's (IEEE): the
squared field of conduction along it, and an estimator without a floor."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as orc  # noqa: E402
from paper_1204_5849_amd import workloads as W  # noqa: E402
from paper_1204_5849_amd.sim import Simulation  # noqa: E402


def _work(ndim, b, **kw):
    tp = 2 * np.pi
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2 if ndim == 3 else 1), bc=(("periodic",) * 2,) * 3)
    base = W.base_keys(0, sd.nbase, ndim)
    return W.Workload(name="range", ndim=ndim, sims=[sd], keys=np.concatenate([base, W.children_of(base[1:2], ndim)]),
                      ic=lambda wl, sim, lv, x, y, z, g: [
                          0.1 + 0.05 * np.sin(tp * (x + y)), 0.05 * np.sin(tp * y), 0.04 * np.cos(tp * x),
                          0.03 * np.sin(tp * (x + y)), b * (1.0 + 0.2 * np.sin(tp * y)), 0.8 * b + 0 * x,
                          0.1 * b + 0 * x, 0.1 + 0.02 * np.sin(tp * x), 0 * x], **kw)


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("b", [1e-153, 4e-155, 1e-158, 1e-163, 0.0])
def test_conduction_along_a_vanishing_field(ndim, b):
    """|B|^2 normal, below 2^-1024 (twice), underflowing to zero, and zero."""
    w = _work(ndim, b, cond="field", kappa0=0.01, kappa_exp=2.5, cond_max_sub=5)
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    A = orc.load_workload(w)
    nsub = A.cfl()[0].nsub
    A.run(1)
    s.advance(1)
    s.sync()
    assert nsub > 1
    leaf = w.leaf_mask()
    g, o = s.state_by_key()[leaf], A.state[leaf]
    z = slice(2, -2) if ndim == 3 else slice(None)
    for k in (0, 1, 2, 3, 7):
        a, c = g[:, k, z, 2:-2, 2:-2], o[:, k, z, 2:-2, 2:-2]
        assert np.isfinite(c).all() and np.abs(a - c).max() <= 1e-11 * np.abs(c).max(), k


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("v", [0.0, 5e-324, 1e-310, 1e-308, 1e-300, 1e-20])
def test_estimate_without_a_floor(ndim, v):
    """eps = 0 and one value near or at zero: the estimate of its block is what
    IEEE division gives, infinity where the quotient overflows."""
    w = _work(ndim, 0.5)
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    at = (int(s.slot_of_key[0]), 0, 2 + 7 if ndim == 3 else 0, 2 + 6, 2 + 5)
    s.U[at] = v
    torch.cuda.synchronize()
    s.fill()
    got = s.estimate([("var", 0, 0.0)])
    p = orc.params_from_workload(w)
    n = (16, 16, 16 if ndim == 3 else 1)
    full = s.state_by_key()
    want = np.array([orc.estimate(p, full[b], n, 0, 0, eps=0.0, level=int(w.keys[b, 1])) for b in range(len(w.keys))])
    assert want[0] > 1e15  # (its smallest value is the planted one)
    fin = np.isfinite(want)
    assert np.array_equal(got[~fin], want[~fin])
    np.testing.assert_allclose(got[fin], want[fin], rtol=1e-12)
