"""The FP32 updates give the bits they gave when golden/fp32_records.txt was
written (by the library as of commit 4fb696d, on an MI355X): the time step after
six cycles of a small tree, an FP64 number formed from the FP32 state, and a
checksum of the leaves.  A different contraction of one product moves both."""
import os
import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1204_5849_amd import workloads as W  # noqa: E402
from paper_1204_5849_amd.sim import Simulation  # noqa: E402

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "fp32_records.txt")


def _ic(wl, sim, lv, x, y, z, g):
    # polynomials and counters only: the same inputs everywhere
    def bump(t):
        return 16.0 * t * t * (1.0 - t) * (1.0 - t)

    n = [1e-3 * W.counter_uniform(11, 0, lv, g, i) for i in range(8)]
    return [1.0 + 0.6 * bump(x) + n[0], 0.8 * bump(y) - 0.3 + n[1], 0.5 * bump(x) - 0.2 + n[2],
            0.3 * bump(z) + n[3], 0.4 + 0.5 * bump(y), 0.3 * bump(z) + n[4], 0.6 * bump(x) - 0.1 + n[5],
            0.3 + 0.2 * bump(y) + n[6], n[7] + 0.0 * x]


def configs():
    for eta in (0.0, 1e-3):
        for rs in ("rusanov", "hllc"):
            for scheme, lim in (("lf", "minmod"), ("lf", "vanleer"), ("lf", "paper"), ("weno", "minmod")):
                yield 3, scheme, lim, rs, eta
        for ndim in (2, 3):
            for lim in ("minmod", "vanleer", "paper"):
                yield ndim, "mmc", lim, "rusanov", eta


def record(ndim, scheme, limiter, riemann, eta):
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2 if ndim == 3 else 1),
                   bc=(("periodic",) * 2, ("outflow",) * 2, ("periodic",) * 2))
    base = W.base_keys(0, sd.nbase, ndim)
    w = W.Workload(name="records", ndim=ndim, sims=[sd],
                   keys=np.concatenate([base, W.children_of(base[1:2], ndim)]), ic=_ic, scheme=scheme,
                   limiter=limiter, riemann=riemann, eta=eta, precision="fp32", glm_mode="fastspeed")
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    s.advance(6)
    s.sync()
    at = torch.from_numpy(s.slot_of_key[w.leaf_mask()].astype(np.int64)).cuda()
    U = s.interior_view()[at].cpu().numpy()
    assert U.dtype == np.float32 and np.isfinite(U).all()
    return float(s.dt[0, 0]).hex(), zlib.crc32(U.tobytes())


def _name(c):
    return " ".join(str(v) for v in c)


@pytest.mark.parametrize("c", list(configs()), ids=_name)
def test_fp32_records(c):
    with open(GOLDEN) as f:
        want = {" ".join(ln.split()[:5]): ln.split()[5:] for ln in f if ln[0] != "#"}
    dt, crc = record(*c)
    assert [dt, f"{crc:08x}"] == want[_name(c)]
