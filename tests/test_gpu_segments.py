"""Row segments of the 2-D update: a small tree's march is split over several
workgroups, a large one's is not.  The same small tree alone and as the first
of many simulations (more and more blocks in one context, so 16, 8, 4, 2 and 1
segments) must give the same state and counters bit for bit, and the oracle's
state to round-off.  The 3-D data-motion passes likewise cut short lists into
more workgroups than long ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as orc  # noqa: E402
from paper_1204_5849_amd import native as N  # noqa: E402
from paper_1204_5849_amd import workloads as W  # noqa: E402
from paper_1204_5849_amd.sim import Simulation  # noqa: E402


def _ic(wl, sim, lv, x, y, z, g):
    tp = 2 * np.pi
    # low pressure and cell-to-cell noise, so that the positivity fall-backs
    # fire (the same noise in every simulation)
    n = [W.counter_uniform(7, 0, lv, g, i) for i in range(4)]
    zero = 0.0 * x
    return [0.3 + 0.25 * n[0], np.sin(tp * y) + n[1], 0.7 * np.cos(tp * x) + n[2], 0.2 + zero,
            0.3 + 0.2 * np.sin(tp * y), 0.2 + zero, 0.1 * np.cos(tp * x), 0.004 + 0.003 * n[3], zero]


def _tree(copies, scheme, eta, riemann, precision):
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 1),
                   bc=(("periodic",) * 2, ("outflow",) * 2, ("periodic",) * 2))
    keys = []
    for s in range(copies):
        base = W.base_keys(s, sd.nbase, 2)
        keys += [base, W.children_of(base[1:2], 2)]  # 7 leaves, coarse-fine faces in x and y
    return W.Workload(name="segments", ndim=2, sims=[sd] * copies, keys=np.concatenate(keys), ic=_ic,
                      scheme=scheme, eta=eta, riemann=riemann, precision=precision)


def _run(w):
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    s.flags()
    s.advance(3)
    s.sync()
    inner = s.state_by_key()[:, :, :, 2:-2, 2:-2]
    return inner, s.flags()[1], s.dt.cpu().numpy()


@pytest.mark.parametrize("scheme,eta,riemann,precision", [("lf", 1e-3, "rusanov", "fp64"),
                                                          ("weno", 0.0, "hllc", "fp64"),
                                                          ("lf", 0.0, "hllc", "fp32"),
                                                          ("weno", 1e-3, "rusanov", "fp32")])
def test_segments_do_not_change_the_update(scheme, eta, riemann, precision):
    N.lib()
    one, cnt, dt = _run(_tree(1, scheme, eta, riemann, precision))
    assert np.isfinite(one).all()
    if precision == "fp64":
        w = _tree(1, scheme, eta, riemann, precision)
        A = orc.load_workload(w)
        A.run(3)
        o = A.state[:, :, :, 2:-2, 2:-2]
        for k in range(8):
            assert np.abs(one[:, k] - o[:, k]).max() <= 1e-11 * np.abs(o[:, k]).max()
    # 14 blocks per workgroup: 40 copies are 20 groups, 80 are 40, 150 are 75, 300 are 150
    for copies in (40, 80, 150, 300):
        many, cm, dm = _run(_tree(copies, scheme, eta, riemann, precision))
        n = len(one)
        for s in (0, copies // 2, copies - 1):
            assert np.array_equal(many[s * n:(s + 1) * n], one), f"{copies} copies, simulation {s}"
        assert np.array_equal(dm, np.repeat(dt, copies, axis=0))
        assert cm == [copies * c for c in cnt]
    assert cnt[1 if scheme == "weno" else 0] > 0


@pytest.mark.parametrize("scheme,precision", [("lf", "fp64"), ("mmc", "fp32")])
def test_short_and_long_lists_3d(scheme, precision):
    """One 3-D tree (a parent, 15 leaves, 7 of them with reflux faces) alone and
    as many copies: 1, 40 and 300 parents, 7 to 2100 reflux leaves, 8 to 2400
    blocks with prolongated ghosts, 7 to 2100 base leaves in the CFL pass."""
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2),
                   bc=(("periodic",) * 2, ("outflow",) * 2, ("periodic",) * 2))

    def tree(copies):
        keys = []
        for s in range(copies):
            base = W.base_keys(s, sd.nbase, 3)
            keys += [base, W.children_of(base[3:4], 3)]
        return W.Workload(name="lists", ndim=3, sims=[sd] * copies, keys=np.concatenate(keys),
                          ic=lambda wl, sim, lv, x, y, z, g: [
                              1 + 0.3 * np.sin(2 * np.pi * (x + z)), 0.4 * np.cos(2 * np.pi * y) + 0 * x,
                              0.3 * np.sin(2 * np.pi * x), 0.2 * np.cos(2 * np.pi * z), 0.5 + 0 * x,
                              0.4 + 0.1 * np.sin(2 * np.pi * y), 0.3 + 0 * x, 0.6 + 0 * x, 0 * x],
                          scheme=scheme, precision=precision, glm_mode="fastspeed")

    def run(w):
        s = Simulation(w, device="cuda:0")
        s.load_initial()
        s.advance(2)
        s.fill()
        s.sync()
        first = np.arange(16)
        last = len(w.keys) - 16 + first
        return s.state_by_key(first), s.state_by_key(last), s.totals()

    one, _, tot = run(tree(1))
    for copies in (40, 300):
        a, b, t = run(tree(copies))
        assert np.array_equal(a, one) and np.array_equal(b, one), copies
        assert np.array_equal(t, np.repeat(tot, copies, axis=0))


@pytest.mark.parametrize("copies,precision", [(1, "fp64"), (1, "fp32"), (25, "fp64"), (25, "fp32"),
                                              (300, "fp32")])
def test_complete_frames_3d(copies, precision):
    """The ghost frames of every block (outflow and periodic edges, prolongated
    ghosts, parents): one variable of a block per item over chunks of blocks,
    against one launch per block, bit for bit.  16 blocks (144 items, 2 per
    XCD), 400 blocks (50 per XCD: chunks of 32 and 16 with a remainder) and
    4800 blocks."""
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2),
                   bc=(("outflow", "outflow"), ("periodic",) * 2, ("outflow",) * 2))
    keys = []
    for s in range(copies):
        base = W.base_keys(s, sd.nbase, 3)
        keys += [base, W.children_of(base[3:4], 3)]
    w = W.Workload(name="frames", ndim=3, sims=[sd] * copies, keys=np.concatenate(keys), ic=_ic,
                   scheme="lf", precision=precision, glm_mode="fastspeed")
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    s.U += torch.rand(s.U.shape, device=s.device, dtype=torch.float64,
                      generator=torch.Generator(s.device).manual_seed(5)).to(s.U.dtype)
    torch.cuda.synchronize()
    ghosts = torch.ones_like(s.U, dtype=torch.bool)
    ghosts[:, :, 2:-2, 2:-2, 2:-2] = False
    base = s.U.clone()
    out = []
    for mode in (N.MAP_LAUNCH_BATCHED, N.MAP_LAUNCH_PER_BLOCK):
        s.U.copy_(base)
        s.U.masked_fill_(ghosts, float("nan"))
        torch.cuda.synchronize()
        s.set_launch(mode)
        s.fill()
        s.sync()
        out.append(s.U.clone())
    assert not out[0].isnan().any()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_complete_frames_3d_where_the_path_changes(precision):
    """Lists up to 4/3 of the CUs are copied in shares of a block, longer ones by
    variable over chunks: 336 and 352 blocks lie on either side with 256 CUs, and
    one block that is its own neighbour takes the most shares."""
    for copies in (21, 22):
        test_complete_frames_3d(copies, precision)
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(1, 1, 1), bc=(("periodic",) * 2,) * 3)
    w = W.Workload(name="frame", ndim=3, sims=[sd], keys=W.base_keys(0, sd.nbase, 3), ic=_ic,
                   scheme="lf", precision=precision, glm_mode="fastspeed")
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    s.fill()
    s.sync()
    u = s.U[0].cpu().numpy()
    inner = u[:, 2:-2, 2:-2, 2:-2]
    assert np.array_equal(u, np.pad(inner, ((0, 0), (2, 2), (2, 2), (2, 2)), mode="wrap"))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_segments_of_a_3d_march(precision):
    """MacCormack with resistivity on one tree (15 leaves, each march in 8
    segments of 2 planes) and on 20, 40 and 150 copies of it: 37 or 38 leaves
    per XCD (32 whole, the others in 4 segments), 75 (11 in 2) and 281 (25
    whole), the same state bit for bit; FP64 to round-off the oracle's."""
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(2, 2, 2),
                   bc=(("periodic",) * 2, ("outflow",) * 2, ("periodic",) * 2))

    def tree(copies):
        keys = []
        for s in range(copies):
            base = W.base_keys(s, sd.nbase, 3)
            keys += [base, W.children_of(base[3:4], 3)]
        return W.Workload(name="marches", ndim=3, sims=[sd] * copies, keys=np.concatenate(keys), eta=1e-3,
                          ic=lambda wl, sim, lv, x, y, z, g: [
                              1 + 0.3 * np.sin(2 * np.pi * (x + z)), 0.4 * np.cos(2 * np.pi * y) + 0 * x,
                              0.3 * np.sin(2 * np.pi * x), 0.2 * np.cos(2 * np.pi * z), 0.5 + 0 * x,
                              0.4 + 0.1 * np.sin(2 * np.pi * y), 0.3 + 0 * x, 0.6 + 0 * x, 0 * x],
                          scheme="mmc", precision=precision, glm_mode="fastspeed")

    def run(copies):
        s = Simulation(tree(copies), device="cuda:0")
        s.load_initial()
        s.advance(2)
        s.sync()
        return s.state_by_key()[:, :, 2:-2, 2:-2, 2:-2]

    one = run(1)
    assert np.isfinite(one).all()
    if precision == "fp64":
        A = orc.load_workload(tree(1))
        A.run(2)
        o = A.state[:, :, 2:-2, 2:-2, 2:-2]
        for k in range(8):
            assert np.abs(one[:, k] - o[:, k]).max() <= 1e-11 * np.abs(o[:, k]).max()
    for copies in (20, 40, 150):
        many = run(copies)
        for s in (0, copies // 2, copies - 1):
            assert np.array_equal(many[s * 16:(s + 1) * 16], one), f"{copies} copies, simulation {s}"


def test_autotune_times_the_update_that_cycles_run():
    """1024 leaves, where the LF update forms the next cycle's CFL maxima and so
    runs whole blocks: the autotuner times that update, which counts a planted
    non-finite cell in each launch, and not the segmented one, which leaves it
    to the CFL pass (one count, of the pass that the autotuner starts with)."""
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(32, 32, 1), bc=(("periodic",) * 2,) * 3)
    w = W.Workload(name="tuned", ndim=2, sims=[sd], keys=W.base_keys(0, sd.nbase, 2), ic=_ic, scheme="lf",
                   precision="fp32")
    s = Simulation(w, device="cuda:0")
    s.load_initial()
    cfg = s.launch_config()
    assert cfg["cfl_in_update_on"] == (1 if len(w.keys) >= 4 * torch.cuda.get_device_properties(0).multi_processor_count else 0)
    s.U[5, 0, 0, 2 + 8, 2 + 8] = float("nan")
    torch.cuda.synchronize()
    s.flags()
    before = s.flags()[1][3]
    s.autotune()
    n = s.flags()[1][3] - before
    assert n > 1 if cfg["cfl_in_update_on"] else n == 1


@pytest.mark.parametrize("ndim,scheme,precision", [(2, "lf", "fp32"), (2, "mmc", "fp64"), (2, "mmc", "fp32"),
                                                   (3, "lf", "fp32"), (3, "lf", "fp64"), (3, "weno", "fp32"),
                                                   (3, "mmc", "fp64"), (3, "mmc", "fp32")])
def test_small_and_uneven_grids(ndim, scheme, precision):
    """Persistent grids that stride (fewer workgroups than work items), below and
    not a multiple of the eight XCDs: the state of the default grid bit for bit."""
    sd = W.SimDesc(lo=(0, 0, 0), hi=(1, 1, 1), nbase=(3, 2, 2 if ndim == 3 else 1),
                   bc=(("periodic",) * 2, ("outflow",) * 2, ("periodic",) * 2))
    keys = []
    for sim in range(8 if ndim == 2 else 3):
        base = W.base_keys(sim, sd.nbase, ndim)
        keys += [base, W.children_of(base[1:2], ndim)]
    w = W.Workload(name="grids", ndim=ndim, sims=[sd] * (8 if ndim == 2 else 3), keys=np.concatenate(keys),
                   ic=_ic, scheme=scheme, eta=1e-3, precision=precision, glm_mode="fastspeed")
    out = []
    for grid in (0, 1, 3, 11, 24):
        s = Simulation(w, device="cuda:0")
        s.load_initial()
        s.set_launch_config(grid_step=grid)
        s.advance(2)
        s.sync()
        inner = slice(2, -2) if ndim == 3 else slice(None)
        out.append((s.state_by_key()[:, :, inner, 2:-2, 2:-2], s.flags()[1]))
    assert np.isfinite(out[0][0]).all()
    for U, cnt in out[1:]:
        assert np.array_equal(U, out[0][0]) and cnt == out[0][1]
