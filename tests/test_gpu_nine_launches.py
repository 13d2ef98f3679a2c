"""The form of an iteration in nine launches: a chain stepped in it next to a
longer one gives what it gives alone in the one-workgroup form, bit for bit, in
every kind of call, and its graphs and launch shapes give what direct launches
give (needs an MI355X).

Each test asks kcm_iteration_launches for the form of its calls, so that a
change of the rule cannot leave the two sides in one form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from gpu_common import TYPES, params  # noqa: E402
from paper_1712_05012_amd import kcm, polyala  # noqa: E402

pytestmark = pytest.mark.gpu

REPORT = ("e_elec", "e_vdw", "e_cav", "max_tau", "max_dtheta", "iterations", "status", "converged")
LONG = 300  # residues of the chain that takes a call into nine launches


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kcm.load_library()


def _chain(m, p, side=False, masked=False, seed=None, types=TYPES):
    seed = 300 + m if seed is None else seed
    th = synth.random_dihedrals(m, seed)
    if side:
        th = np.concatenate([th, synth.random_chi(m, seed)])
    mask = np.ones(th.size, np.uint8)
    if masked:
        mask[::7] = 0
    return kcm.Chain(synth.sequence(m, seed), types, p, theta0=th, joint_mask=mask, side_chains=side)


def _form(launches, *chains):
    assert kcm.kcm_iteration_launches([c.n_atoms // 10 for c in chains]) == launches


def _same(a, b):
    for x, y in ((a.state(), b.state()), (a.atom_terms(), b.atom_terms()), (a.cells(), b.cells())):
        for k in x:
            assert np.array_equal(x[k], y[k]), k


def _free(*chains):
    for c in chains:
        c.free()


# around the sizes of a workgroup (256, 512, 768 atoms) and of the longest chain
# that takes the one-workgroup form in any call (2,048 atoms)
@pytest.mark.parametrize("m", [1, 2, 25, 26, 51, 52, 76, 77, 102, 153, 204])
@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_step_reports_and_states(precision, m):
    p, side = params(precision), m % 2 == 0
    a, b, other = _chain(m, p, side, True), _chain(m, p, side, True), _chain(LONG, p)
    _form(2, a)
    _form(9, b, other)
    print(f"case=nine precision={precision} m={m} side={side}", flush=True)
    for n_iter in (1, 3):
        _, ra = kcm.kcm_step([a], n_iter, check=False)
        _, rb = kcm.kcm_step([b, other], n_iter, check=False)
        assert all(getattr(ra[0], f) == getattr(rb[0], f) for f in REPORT)
        _same(a, b)
    # a chain goes from one form to the other and back
    kcm.kcm_step([a, other], 2)
    kcm.kcm_step([b], 2)
    _same(a, b)
    kcm.kcm_step([a], 1)
    kcm.kcm_step([b, other], 1)
    _same(a, b)
    _free(a, b, other)


def test_long_chains_in_the_one_workgroup_form():
    # chains past 2,048 atoms, up to the longest that a workgroup holds, in a
    # call of many; alone or next to a longer one they take nine launches
    p = params(kcm.KCM_MIXED)
    sizes = [640, 512, 333, 205, 154, 77]
    many = [_chain(m, p, m == 333, True) for m in sizes]
    many += [_chain(640, p, seed=7) for _ in range(122)]
    _form(2, *many)
    print(f"case=nine-long chains={len(many)}", flush=True)
    _, reps = kcm.kcm_step(many, 2, check=False)
    other = _chain(641, p)
    for m, c, r in zip(sizes, many, reps):
        alone = _chain(m, p, m == 333, True)
        _form(9, alone, other)
        _, ra = kcm.kcm_step([alone, other], 2, check=False)
        assert all(getattr(ra[0], f) == getattr(r, f) for f in REPORT)
        _same(alone, c)
        alone.free()
    _free(other, *many)


@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_failures_stop_the_same_chain(precision):
    p = params(precision)
    huge = synth.ResidueTypes(q=TYPES.q * 1e300, sigma=TYPES.sigma, eps=TYPES.eps, hydro=TYPES.hydro)
    a = [_chain(20, p), _chain(4, p, types=huge), _chain(30, p, True)]
    b = [_chain(20, p), _chain(4, p, types=huge), _chain(30, p, True)]
    other = _chain(LONG, p)
    _form(2, *a)
    _form(9, other, *b)
    print(f"case=nine-failures precision={precision}", flush=True)
    angles = [c.theta() for c in a]
    angles[0][5] = np.nan  # no grid: stops before its first iteration
    held = [kcm.kcm_set_theta_batch(a, angles), kcm.kcm_set_theta_batch(b, angles)]
    _, ra = kcm.kcm_step(a, 3, check=False)
    _, rb = kcm.kcm_step([other] + b, 3, check=False)
    assert [r.status for r in ra] == [kcm.KCM_E_NUMERIC, kcm.KCM_E_NUMERIC, kcm.KCM_OK]
    assert [r.iterations for r in ra] == [0, 0, 3]
    for x, y in zip(ra, rb[1:]):
        assert (x.status, x.iterations, x.converged) == (y.status, y.iterations, y.converged)
    assert rb[0].status == 0 and rb[0].iterations == 3
    _same(a[2], b[2])
    # a failed chain stays stopped, and fresh angles start it again
    _, ra = kcm.kcm_step(a, 1, check=False)
    _, rb = kcm.kcm_step([other] + b, 1, check=False)
    assert [r.iterations for r in ra] == [r.iterations for r in rb[1:]] == [0, 0, 4]
    angles[0] = synth.random_dihedrals(20, 9)
    held += [kcm.kcm_set_theta_batch([a[0]], angles[:1]), kcm.kcm_set_theta_batch([b[0], other], [angles[0], other.theta()])]
    kcm.kcm_step(a[:1], 2)
    kcm.kcm_step([b[0], other], 2)
    _same(a[0], b[0])
    _free(other, *a, *b)
    del held


def test_limits_and_folds_stop_at_the_same_iteration():
    p = params(kcm.KCM_MIXED)
    a, b, other = [_chain(20 + k, p) for k in range(4)], [_chain(20 + k, p) for k in range(4)], _chain(LONG, p)
    _form(2, *a)
    _form(9, other, *b)
    print("case=nine-limits", flush=True)
    for set_ in (a, b):
        kcm.kcm_set_limits(set_[0].handle, 0.0, 7)    # an iteration cap
        kcm.kcm_set_limits(set_[1].handle, 10.0, 0)   # converges on its first step
    _, ra = kcm.kcm_step(a, 9)
    _, rb = kcm.kcm_step([other] + b, 9)
    assert [r.iterations for r in ra] == [7, 1, 9, 9] and [r.converged for r in ra] == [0, 1, 0, 0]
    for x, y in zip(ra, rb[1:]):
        assert all(getattr(x, f) == getattr(y, f) for f in REPORT)
    # a fold suspends the chains' own limits; its steps are at most max_step (1e-3), so 2e-3 ends it at once
    for tol, cap, every in ((1e-30, 8, 3), (2e-3, 8, 3)):
        _, fa = kcm.kcm_fold(a, tol, cap, every)
        _, fb = kcm.kcm_fold([other] + b, tol, cap, every)
        for x, y in zip(fa, fb[1:]):
            assert (x.iterations, x.converged, x.status) == (y.iterations, y.converged, y.status)
        assert {x.iterations for x in fa} == ({8} if tol < 1e-3 else {1})
    for x, y in zip(a, b):
        _same(x, y)
    _free(other, *a, *b)


@pytest.mark.parametrize("terms", [kcm.KCM_TERM_ALL, kcm.KCM_TERM_ELEC | kcm.KCM_TERM_VDW])
def test_monte_carlo_minimization(terms):
    p = polyala.experiment_params(terms == kcm.KCM_TERM_ALL, kcm.KCM_FP64)
    spec = [(9, False), (14, True)]
    a, b = ([_chain(m, p, side, True) for m, side in spec] for _ in range(2))
    other = _chain(LONG, p)
    _form(2, *a)
    _form(9, other, *b)
    print(f"case=nine-mc terms={terms}", flush=True)
    moves = [synth.mc_moves(4, c.n_joints, 70 + k) for k, c in enumerate([other] + a)]
    delta, u = [d for d, _ in moves], np.stack([v for _, v in moves])
    _, ra = kcm.kcm_mc_minimize(a, delta[1:], u[1:], 3, 1.0)
    _, rb = kcm.kcm_mc_minimize([other] + b, delta, u, 3, 1.0)
    for x, y, ca, cb in zip(ra, rb[1:], a, b):
        for f in ("e_start", "e_accepted", "e_best", "trials", "accepted", "status"):
            assert getattr(x, f) == getattr(y, f), f
        assert np.array_equal(ca.mc_best_theta(), cb.mc_best_theta())
        _same(ca, cb)
    # and on from the accepted angles
    _, ra = kcm.kcm_step(a, 2)
    _, rb = kcm.kcm_step([other] + b, 2)
    for x, y, ca, cb in zip(ra, rb[1:], a, b):
        assert all(getattr(x, f) == getattr(y, f) for f in REPORT)
        _same(ca, cb)
    _free(other, *a, *b)


@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_noalloc_step_equals_kcm_step(precision):
    # several chains: without maps of workgroups to chains each kernel searches
    p = params(precision)
    sizes = (7, LONG, 120, 15, 260)
    a, b = [_chain(m, p, m == 15) for m in sizes], [_chain(m, p, m == 15) for m in sizes]
    print(f"case=nine-noalloc precision={precision}", flush=True)
    for idx, n_iter in (([0, 1, 2, 3, 4], 3), ([1, 3], 2), ([4], 1)):
        _form(9, *[a[i] for i in idx])
        _, ra = kcm.kcm_step([a[i] for i in idx], n_iter)
        _, rb = kcm.kcm_step_noalloc([b[i] for i in idx], n_iter)
        for i, x, y in zip(idx, ra, rb):
            assert all(getattr(x, f) == getattr(y, f) for f in REPORT), i
            _same(a[i], b[i])
    _free(*a, *b)


@pytest.mark.parametrize("depth", [1, 4])
def test_graph_replay_equals_direct_launches(depth):
    # replays (one iteration a graph, or four and single ones for the rest of a
    # call) with eager work, synchronisations and another set's graph between
    # them, against direct launches after every call
    p = params(kcm.KCM_MIXED)
    sizes = (LONG, 27, 14)
    a, b, c = ([_chain(m, p, m == 14) for m in sizes] for _ in range(3))
    _form(9, *a)
    print(f"case=nine-graphs depth={depth}", flush=True)
    try:
        for rep in range(4):
            kcm.kcm_set_graphs(depth)
            kcm.kcm_step(a, 3 + 3 * rep)
            assert torch.ones(1000, device="cuda").sum().item() == 1000.0
            kcm.kcm_step(c[:2], depth)
            kcm.kcm_set_graphs(0)
            kcm.kcm_step(b, 3 + 3 * rep)
            torch.cuda.synchronize()
            for x, y in zip(a, b):
                _same(x, y)
    finally:
        kcm.kcm_set_graphs(1)
        _free(*a, *b, *c)


def test_force_kernel_shapes():
    # past the 2,048 atoms from which the orders of the atoms over the XCDs
    # differ; each shape and precision captures its own graph of a set
    sizes = (LONG, 9, 120)
    ref = {}
    try:
        for v in (0, 1, 2, 3, 0):
            kcm.kcm_set_force_variant(v)
            for prec in (kcm.KCM_MIXED, kcm.KCM_FP64):
                cs = [_chain(m, params(prec), m == 9) for m in sizes]
                _form(9, *cs)
                print(f"case=nine-shapes shape={v} precision={prec}", flush=True)
                kcm.kcm_step(cs, 3)
                for w in ((v + 1) % kcm.KCM_FORCE_VARIANTS, v):  # the same set's graph in another shape
                    kcm.kcm_set_force_variant(w)
                    kcm.kcm_step(cs, 1)
                states = [c.state() for c in cs]
                for x, y in zip(states, ref.setdefault(prec, states)):
                    for k in x:
                        assert np.array_equal(x[k], y[k]), (v, prec, k)
                _free(*cs)
    finally:
        kcm.kcm_set_force_variant(0)


def test_more_sets_with_graphs_than_a_stream_keeps():
    # six sets in turn, four of them with a captured graph; one of these is
    # freed and built again, and each is met again after its table was given up
    p = params(kcm.KCM_MIXED)
    spec = [[LONG, 3], [30], [250, 7], [LONG + 10], [12, 260], [26, 5]]
    sets = [[_chain(m, p, seed=100 * k + i) for i, m in enumerate(ms)] for k, ms in enumerate(spec)]
    assert [kcm.kcm_iteration_launches(ms) for ms in spec] == [9, 2, 9, 9, 9, 2]
    print("case=nine-sets", flush=True)
    for turn in range(3):
        for k in (0, 1, 2, 3, 4, 5, 2, 0):
            kcm.kcm_step(sets[k], 1 + turn)
        if turn == 0:
            _free(*sets[2])
            sets[2] = [_chain(m, p, seed=900 + i) for i, m in enumerate(spec[2])]
    its = [12, 6, 10, 6, 6, 6]
    try:
        kcm.kcm_set_graphs(0)
        for k, ms in enumerate(spec):
            for i, m in enumerate(ms):
                alone = _chain(m, p, seed=900 + i if k == 2 else 100 * k + i)
                kcm.kcm_step([alone], its[k])
                _same(alone, sets[k][i])
                alone.free()
    finally:
        kcm.kcm_set_graphs(1)
        for s in sets:
            _free(*s)


@pytest.mark.parametrize("sizes,launches", [((12,), 2), ((30, 7, 90), 2), ((LONG, 7), 9)])
def test_noalloc_step_in_a_callers_graph(sizes, launches):
    # a caller's own capture of kcm_step_noalloc, replayed with eager work and
    # synchronisations between, against kcm_step
    p = params(kcm.KCM_MIXED)
    a, b = [_chain(m, p, m == 7) for m in sizes], [_chain(m, p, m == 7) for m in sizes]
    _form(launches, *a)
    print(f"case=nine-capture sizes={sizes}", flush=True)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        kcm.kcm_step_noalloc(b, 1, report=False)  # the table of the set is there before the capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            kcm.kcm_step_noalloc(b, 2, report=False)
    kcm.kcm_step(a, 1)
    for k in range(4):
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        assert torch.ones(1000, device="cuda").sum().item() == 1000.0
        kcm.kcm_step(a, 2)
        for x, y in zip(a, b):
            _same(x, y)
    _free(*a, *b)
