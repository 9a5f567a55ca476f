"""Non-finite values stay visible: a NaN beside finite cells does to their slopes
what it does in the oracle, and to the speeds of their faces what a comparison
leaves of it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as orc  # noqa: E402
from paper_1204_5849_amd import workloads as W  # noqa: E402
from paper_1204_5849_amd.sim import Simulation  # noqa: E402


def _ic(wl, sim, lv, x, y, z, g):
    tp = 2 * np.pi
    return [1.0 + 0.3 * np.sin(tp * x) * np.cos(tp * y), 0.4 * np.sin(tp * y), 0.3 * np.sin(tp * (x + z)),
            0.1 * np.cos(tp * z), 0.5 + 0.2 * np.cos(tp * y), 0.3 * np.sin(tp * x),
            0.2 + 0.1 * np.sin(tp * z), 1.0 + 0.2 * np.cos(tp * x), 0.05 * np.sin(tp * y)]


def _work(ndim, ic=_ic, **kw):
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2 if ndim == 3 else 1), bc=(("periodic",) * 2,) * 3)
    return W.Workload(name="nonfinite", ndim=ndim, sims=[sd], keys=W.base_keys(0, sd.nbase, ndim), ic=ic,
                      glm_mode="fastspeed", **kw)


def _inside(U):
    return U[:, :, 2:-2, 2:-2, 2:-2] if U.shape[2] > 1 else U[:, :, :, 2:-2, 2:-2]


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("scheme,var", [("lf", 8), ("mmc", 0), ("mmc", 5), ("mmc", 8)])
def test_nan_beside_finite_cells(ndim, scheme, var):
    w = _work(ndim, scheme=scheme, limiter="minmod")
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    A = orc.load_workload(w)
    recs = A.cfl()
    s.cfl()
    cell = (0, var, 2 + 7 if ndim == 3 else 0, 2 + 6, 2 + 5)
    A.state[cell] = np.nan
    s.sync()
    s.U[(int(s.slot_of_key[0]),) + cell[1:]] = float("nan")
    out = torch.zeros_like(s.U)
    torch.cuda.synchronize()
    s.step(out)
    s.sync()
    A.fill()
    A.step(recs)
    g, o = _inside(out.cpu().numpy()[s.slot_of_key]), _inside(A.state)
    assert np.isnan(o).any() and not np.isnan(o).all()
    assert np.array_equal(np.isnan(g), np.isnan(o))
    for k in range(9):
        fin = np.isfinite(o[:, k])
        assert np.abs(g[:, k] - o[:, k])[fin].max() <= 1e-11 * max(1.0, np.abs(o[:, k][fin]).max()), k
    assert list(s.flags()[1][:2]) == list(A.counters()[:2])


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("riemann", ["rusanov", "hllc"])
def test_nan_field_reaches_the_density(ndim, precision, riemann):
    """A NaN in B_y of one cell makes its fast speed NaN.  The larger speed of a
    face is the right one unless the left one is larger, so the faces on whose
    right the cell lies have NaN fluxes in every variable: the density of the
    cell and of its lower neighbours is NaN."""
    w = _work(ndim, scheme="lf", riemann=riemann, precision=precision)
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    s.cfl()
    s.sync()
    z, y, x = 2 + 7 if ndim == 3 else 0, 2 + 6, 2 + 5
    b = int(s.slot_of_key[0])
    s.U[b, 5, z, y, x] = float("nan")
    out = torch.zeros_like(s.U)
    torch.cuda.synchronize()
    s.step(out)
    s.sync()
    rho = out[b, 0]
    cells = [rho[z, y, x], rho[z, y, x - 1], rho[z, y - 1, x]] + ([rho[z - 1, y, x]] if ndim == 3 else [])
    assert all(bool(c.isnan()) for c in cells)
    s.U.copy_(out)
    torch.cuda.synchronize()
    s.cfl()
    assert s.flags()[1][3] > 0
