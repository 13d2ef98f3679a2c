"""The one-workgroup form of the iteration (k_chain and the force kernel) and
the form in nine launches give the same results bit for bit (needs an MI355X).

A call takes the one-workgroup form when its largest chain is short or its
chains are many; the same chain stepped next to a longer one takes the other.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from gpu_common import TYPES, params  # noqa: E402
from paper_1712_05012_amd import kcm  # noqa: E402

pytestmark = pytest.mark.gpu

REPORT = ("e_elec", "e_vdw", "e_cav", "max_tau", "max_dtheta", "iterations", "status", "converged")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kcm.load_library()


def _chain(m, p, side_chains):
    th = synth.random_dihedrals(m, 40 + m)
    if side_chains:
        th = np.concatenate([th, synth.random_chi(m, 40 + m)])
    mask = np.ones(th.size, np.uint8)
    mask[::7] = 0
    return kcm.Chain(synth.sequence(m, 40 + m), TYPES, p, theta0=th, joint_mask=mask, side_chains=side_chains)


def _same(a, b):
    sa, sb, ca, cb = a.state(), b.state(), a.cells(), b.cells()
    for k in sa:
        assert np.array_equal(sa[k], sb[k]), k
    for k in ca:
        assert np.array_equal(ca[k], cb[k]), k


# around the sizes of a workgroup (256, 512, 768 atoms) and of the longest
# chain that takes the form in any call (1,536 atoms)
@pytest.mark.parametrize("m", [1, 2, 25, 26, 51, 52, 76, 77, 102, 103, 153])
@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_short_chain_alone_equals_next_to_a_long_one(precision, m):
    side = m % 2 == 0
    p = params(precision)
    a, b, other = _chain(m, p, side), _chain(m, p, side), _chain(200, p, False)
    print(f"case=chain-form precision={precision} m={m} side={side}", flush=True)
    for n_iter in (1, 3):
        _, ra = kcm.kcm_step([a], n_iter, check=False)
        _, rb = kcm.kcm_step([b, other], n_iter, check=False)
        assert all(getattr(ra[0], f) == getattr(rb[0], f) for f in REPORT)
        _same(a, b)
    for c in (a, b, other):
        c.free()


def test_long_chains_among_many_equal_the_same_alone():
    p = params(kcm.KCM_MIXED)
    sizes = [640, 154, 205, 333, 512] + [3] * 123
    many = [_chain(m, p, m == 333) for m in sizes]
    print(f"case=chain-form chains={len(many)}", flush=True)
    kcm.kcm_step(many, 2)
    for m, c in zip(sizes[:5], many):
        alone = _chain(m, p, m == 333)
        kcm.kcm_step([alone], 2)
        _same(alone, c)
        alone.free()
    for c in many:
        c.free()


def test_conformation_without_a_grid_stops_the_chain_in_both_forms():
    p = params(kcm.KCM_FP64)
    a, b, other = _chain(20, p, False), _chain(20, p, False), _chain(200, p, False)
    bad = a.theta()
    bad[5] = np.nan
    print("case=chain-form non-finite angle", flush=True)
    held = [kcm.kcm_set_theta_batch([c], [bad]) for c in (a, b)]
    _, ra = kcm.kcm_step([a], 2, check=False)
    _, rb = kcm.kcm_step([b, other], 2, check=False)
    assert ra[0].status == rb[0].status == kcm.KCM_E_NUMERIC
    assert ra[0].iterations == rb[0].iterations == 0
    assert rb[1].status == 0 and rb[1].iterations == 2
    # fresh angles start it again
    good = synth.random_dihedrals(20, 9)
    held += [kcm.kcm_set_theta_batch([c], [good]) for c in (a, b)]
    kcm.kcm_step([a], 2)
    kcm.kcm_step([b, other], 2)
    _same(a, b)
    for c in (a, b, other):
        c.free()
    del held
