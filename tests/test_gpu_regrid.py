"""GPU parity of the regrid path (paper Sec. 4.5) against the oracle: the
error estimator per block, the state moved onto a new tree (copies,
prolongation of new blocks, restriction, fill), and cycles after a regrid."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle.regrid import regrid as oracle_regrid  # noqa: E402
from paper_1204_5849_amd import native as N  # noqa: E402
from paper_1204_5849_amd import workloads as W  # noqa: E402
from tests.helpers import rel_linf  # noqa: E402

CRIT = [("var", 0, 1e-12), ("bmag", 0, 0.1)]


def _say(msg):
    print(f"[gpu-regrid] {msg}", flush=True)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    N.lib()
    return "cuda:0"


def _sim(w, **kw):
    from paper_1204_5849_amd.sim import Simulation
    s = Simulation(w, **kw)
    s.load_initial()
    return s


def _oracle_err(orc, w, U):
    p = orc.params_from_workload(w)
    n3 = (16, 16, 16) if w.ndim == 3 else (16, 16, 1)
    out = np.zeros(len(w.keys))
    for b in range(len(w.keys)):
        lv = int(w.keys[b, 1])
        t = np.ascontiguousarray(U[b])
        out[b] = max(orc.estimate(p, t, n3, 0, 0, eps=1e-12, level=lv),
                     orc.estimate(p, t, n3, 1, 0, eps=0.1, level=lv))
    return out


def _workload(name, precision):
    if name == "blast":
        return W.blast3d(nbase=2, levels=2, precision=precision)
    return W.harris3d(nbase=2, levels=3, precision=precision)


def _tree2d(precision):
    """Orszag-Tang on an 8 x 8 base with the left half refined once."""
    base = W.orszag_tang(8)
    keys = base.keys
    kids = W.children_of(keys[(keys[:, 2] < 4)], 2)
    return W.ot_amr(np.concatenate([keys, kids]), nbase=8, precision=precision)


@pytest.mark.parametrize("name,precision", [("ot", "fp64"), ("ot", "fp32"), ("blast", "fp64"),
                                            ("harris", "fp32")])
def test_estimate_matches_oracle(dev, orc, name, precision):
    """The estimator after two cycles (ghost frames left as the cycle leaves
    them: the estimate reads in place) against the oracle's estimate of its
    own state after the same two cycles.  FP64: the states agree to rounding,
    so the estimates to 1e-10 relative (1e-13 absolute below 1e-3, where
    smooth blocks estimate 0); FP32: the state itself differs from the FP64
    one by FP32 rounding, 1e-4 relative (1e-6 absolute)."""
    w = _tree2d(precision) if name == "ot" else _workload(name, precision)
    _say(f"estimate {name} {precision}: {len(w.keys)} blocks")
    s = _sim(w)
    s.advance(2)
    got = s.estimate(CRIT)
    A = orc.load_workload(w)
    A.run(2)
    want = _oracle_err(orc, w, A.state)
    big = want > 1e-3
    rel = np.abs(got - want)[big] / want[big]
    small = np.abs(got - want)[~big].max() if (~big).any() else 0.0
    _say(f"  max rel diff {rel.max():.2e} over {int(big.sum())} blocks, max abs diff "
         f"{small:.2e} over the others, estimates in [{want.min():.3g}, {want.max():.3g}]")
    assert big.sum() >= 8
    assert rel.max() <= (1e-10 if precision == "fp64" else 1e-4)
    assert small <= (1e-13 if precision == "fp64" else 1e-6)


def _interior(w, U):
    if w.ndim == 3:
        return U[:, :, 2:-2, 2:-2, 2:-2]
    return U[:, :, :, 2:-2, 2:-2]


def _gap_threshold(vals, lo, hi):
    """A threshold between two sorted distinct values at positions in
    [lo, hi) of the sorted list, at the largest relative gap there, so that
    estimates that differ by rounding fall on the same side of it."""
    v = np.sort(np.unique(vals))
    if len(v) < 2:  # all alike: every one of them is above the threshold
        return v[0] * (1.0 - 1e-6)
    a = min(max(1, int(lo * len(v))), len(v) - 1)
    b = min(max(a + 1, int(hi * len(v))), len(v))
    i = max(range(a, b), key=lambda j: (v[j] - v[j - 1]) / v[j])
    return 0.5 * (v[i] + v[i - 1])


def _thresholds(w, err):
    """Refine about the top fifth of the leaves; destroy the children of
    about the smoother half of the blocks whose children are all leaves."""
    leaves = w.leaf_mask()
    tr = _gap_threshold(err[leaves], 0.7, 0.9)
    keyset = {tuple(int(v) for v in k) for k in w.keys}
    kid_parents = {(s2, l2 - 1, x2 >> 1, y2 >> 1, z2 >> 1) for (s2, l2, x2, y2, z2) in keyset}
    cand = []
    for i, k in enumerate(w.keys):
        if leaves[i]:
            continue
        s, lv, x, y, z = (int(v) for v in k)
        kids = [(s, lv + 1, 2 * x + (c & 1), 2 * y + ((c >> 1) & 1),
                 2 * z + ((c >> 2) & 1) if w.ndim == 3 else 0) for c in range(1 << w.ndim)]
        if all(c in keyset and c not in kid_parents for c in kids):
            cand.append(err[i])
    if len(np.unique(cand)) > 1:
        tc = _gap_threshold(cand, 0.3, 0.7)
    else:  # all candidates alike (a symmetric problem): all of them qualify
        tc = max(cand) * (1.0 + 1e-6) + 1e-300
    return tr, tc


def _changes(w_old, w_new):
    old = {tuple(int(v) for v in k) for k in w_old.keys}
    new = {tuple(int(v) for v in k) for k in w_new.keys}
    return len(new - old), len(old - new)


def _oracle_remap(orc, w_new, w_old, old_full):
    p = orc.params_from_workload(w_new)
    B = orc.Amr(p, 16, w_new.sims, w_new.keys)
    old_index = {tuple(int(v) for v in k): i for i, k in enumerate(w_old.keys)}
    new_blocks = []
    for i, k in enumerate(w_new.keys):
        j = old_index.get(tuple(int(v) for v in k))
        if j is None:
            new_blocks.append(i)
        else:
            B.state[i] = old_full[j]
    B.fill()
    for i in new_blocks:
        B.prolong_block(i)
    B.restrict()
    B.fill()
    return B, new_blocks


@pytest.mark.parametrize("name,cycles", [("ot", 0), ("blast", 2)])
def test_remap_matches_oracle(dev, orc, name, cycles):
    """One regrid, decided and carried out by each side on its own state:
    the oracle forms its estimates, thresholds and new tree (oracle.regrid)
    and moves its state (copies, prolongation, restriction, fill); the
    library's estimate, tree edit with the same thresholds and remap must
    give the same tree and the same state: bit for bit from the initial
    data (Orszag-Tang), to 1e-11 after two cycles (the blast, whose initial
    density and field are uniform, so that every estimate is zero)."""
    # 3-D: a 4^3 base, so that smooth blocks can lose their children without
    # touching the new finest blocks (on a 2^3 periodic base every block
    # touches every other)
    w = _tree2d("fp64") if name == "ot" else W.blast3d(nbase=4, levels=2, precision="fp64")
    A = orc.load_workload(w)
    A.run(cycles)
    err_o = _oracle_err(orc, w, A.state)
    tr, tc = _thresholds(w, err_o)
    want_keys = oracle_regrid([tuple(int(v) for v in k) for k in w.keys], w.sims, w.ndim,
                              {tuple(int(v) for v in k): e for k, e in zip(w.keys, err_o)},
                              tr, tc, 3)
    s = _sim(w)
    s.advance(cycles)
    new = s.regrid(CRIT, tr, tc, 3)
    assert [tuple(int(v) for v in k) for k in new.wl.keys] == want_keys
    B, new_blocks = _oracle_remap(orc, new.wl, w, A.state)
    created, destroyed = _changes(w, new.wl)
    _say(f"remap {name}: {len(w.keys)} -> {len(new.wl.keys)} blocks, {created} created, "
         f"{destroyed} destroyed (tau_refine {tr:.3g}, tau_coarsen {tc:.3g})")
    assert created == len(new_blocks) and created > 0 and destroyed > 0
    got = new.state_by_key()
    if cycles == 0:
        assert np.array_equal(got, B.state)
    else:
        err = rel_linf(_interior(new.wl, got), _interior(new.wl, B.state))
        _say(f"  rel Linf per var {np.array2string(err, precision=2)}")
        assert np.all(err[:8] <= 1e-11)


@pytest.mark.parametrize("name", ["ot", "blast"])
def test_regrid_then_cycles_match_oracle(dev, orc, name):
    """Cycles, a regrid that refines and coarsens, more cycles, each side on
    its own state: the oracle's estimates decide the thresholds and its own
    tree, which the library's tree edit must reproduce; the leaves then agree
    with the oracle (FP64)."""
    w = _tree2d("fp64") if name == "ot" else _workload(name, "fp64")
    s = _sim(w)
    A = orc.load_workload(w)
    s.advance(3)
    A.run(3)
    err_o = _oracle_err(orc, w, A.state)
    tr, tc = _thresholds(w, err_o)
    want_keys = oracle_regrid([tuple(int(v) for v in k) for k in w.keys], w.sims, w.ndim,
                              {tuple(int(v) for v in k): e for k, e in zip(w.keys, err_o)},
                              tr, tc, 3)
    new = s.regrid(CRIT, tr, tc, 3)
    assert [tuple(int(v) for v in k) for k in new.wl.keys] == want_keys
    B, _ = _oracle_remap(orc, new.wl, w, A.state)
    new.advance(4)
    B.run(4)
    leaves = new.wl.leaf_mask()
    g = _interior(new.wl, new.state_by_key()[leaves])
    o = _interior(new.wl, B.state[leaves])
    err8 = rel_linf(g, o)
    created, destroyed = _changes(w, new.wl)
    _say(f"{name} regrid ({created} created, {destroyed} destroyed) + 4 cycles: "
         f"rel Linf per var {np.array2string(err8, precision=2)}")
    assert created > 0
    assert np.all(err8[:8] <= 1e-11)


def test_run_adaptive_equals_manual_regrids(dev):
    """Regrids inside the run at the Sec. 4.5 interval, re-planned in place:
    the same cycles and regrids done by hand with new contexts give the same
    trees and, bit for bit, the same state; once both buffer pairs have held
    a tree, the regrids reuse them."""
    w = _tree2d("fp64")
    a = _sim(w)
    err0 = a.estimate(CRIT)
    tr, tc = _thresholds(w, err0)
    log = a.run_adaptive(9, CRIT, tr, tc, 3, c_r=0.1)
    _say(f"adaptive run: regrids at {log}")
    assert len(log) >= 3
    ptrs = []
    b = _sim(w)
    done = 0
    for cyc, nb in log:
        b.graph_run(cyc - done)
        done = cyc
        b = b.regrid(CRIT, tr, tc, 3)
        assert len(b.wl.keys) == nb
    b.graph_run(9 - done)
    assert np.array_equal(a.wl.keys, b.wl.keys)
    a.fill()
    b.fill()
    assert np.array_equal(a.state_by_key(), b.state_by_key())
    # two more regrids in place: the state buffers alternate between two pairs
    for _ in range(2):
        a.regrid_in_place(CRIT, tr, tc, 3)
        ptrs.append(a._ubuf.data_ptr())
    a.regrid_in_place(CRIT, tr, tc, 3)
    assert a._ubuf.data_ptr() == ptrs[0]


@pytest.mark.parametrize("name,precision", [("ot", "fp64"), ("blast", "fp32"), ("harris", "fp64")])
def test_criteria_together_equal_criteria_alone(dev, name, precision):
    """1 to 4 criteria in one pass: the maximum of the passes of each alone, bit for bit."""
    w = _tree2d(precision) if name == "ot" else _workload(name, precision)
    s = _sim(w)
    s.advance(2)
    crit = [("bmag", 0, 0.1), ("var", 7, 1e-12), ("var", 1, 0.3), ("var", 0, 1e-12)]
    alone = [s.estimate([c], xi=0.5) for c in crit]
    for n in range(2, 5):
        assert np.array_equal(s.estimate(crit[:n], xi=0.5), np.maximum.reduce(alone[:n]))
