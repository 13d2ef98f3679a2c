"""The force kernel without the solvation term gives what the general one gives,
bit for bit (needs an MI355X).

A call whose chains all lack the term takes the kernel that has no neighbour
list; the same chain next to one that has it takes the general kernel.
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


def _chain(m, p):
    return kcm.Chain(synth.sequence(m, 70 + m), TYPES, p, theta0=synth.random_dihedrals(m, 70 + m))


# fewer candidates than a wave, around one and several trips of 64, chains of
# both forms of the iteration, and around 2,048 atoms (the groups in which the
# atoms go to the compute dies)
@pytest.mark.parametrize("m", [1, 6, 7, 13, 26, 77, 200, 204, 205, 410])
@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_pair_terms_alone_equal_next_to_a_solvated_chain(precision, m):
    pair, full = params(precision, terms=kcm.KCM_TERM_ELEC | kcm.KCM_TERM_VDW), params(precision)
    a, b, other = _chain(m, pair), _chain(m, pair), _chain(5, full)
    print(f"case=force-terms precision={precision} m={m}", flush=True)
    for n_iter in (1, 3):
        _, ra = kcm.kcm_step([a], n_iter, check=False)
        _, rb = kcm.kcm_step([b, other], n_iter, check=False)
        assert all(getattr(ra[0], f) == getattr(rb[0], f) for f in REPORT)
        sa, sb = a.state(), b.state()
        for k in sa:
            assert np.array_equal(sa[k], sb[k]), k
    assert ra[0].e_cav == 0.0
    for c in (a, b, other):
        c.free()


@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_no_terms_at_all(precision):
    c = _chain(30, params(precision, terms=0))
    print(f"case=force-terms none precision={precision}", flush=True)
    _, r = kcm.kcm_step([c], 1)
    assert (r[0].e_elec, r[0].e_vdw, r[0].e_cav, r[0].max_tau) == (0.0, 0.0, 0.0, 0.0)
    assert not np.any(c.state()["force"])
    c.free()
