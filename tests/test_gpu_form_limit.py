"""Chains up to and just past the longest that takes the one-workgroup form in
any call (2,048 atoms) give in it what the form in nine launches gives, bit for
bit (needs an MI355X): alone, and next to a chain too long for it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from gpu_common import TYPES, params  # noqa: E402
from paper_1712_05012_amd import kcm  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kcm.load_library()


def _chain(m, p, side_chains=False):
    th = synth.random_dihedrals(m, 30 + m)
    if side_chains:
        th = np.concatenate([th, synth.random_chi(m, 30 + m)])
    return kcm.Chain(synth.sequence(m, 30 + m), TYPES, p, theta0=th, side_chains=side_chains)


@pytest.mark.parametrize("m,side", [(5, True), (25, True), (26, False), (60, True), (154, False), (180, True), (204, False), (205, False)])
@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_one_workgroup_equals_nine_launches(precision, m, side):
    p = params(precision)
    a, b, other = _chain(m, p, side), _chain(m, p, side), _chain(300, p)
    print(f"case=form-limit precision={precision} m={m} side={side}", flush=True)
    for n_iter in (1, 2):
        kcm.kcm_step([a], n_iter, check=False)
        kcm.kcm_step([b, other], n_iter, check=False)
        sa, sb, ca, cb = a.state(), b.state(), a.cells(), b.cells()
        for k in sa:
            assert np.array_equal(sa[k], sb[k]), k
        for k in ca:
            assert np.array_equal(ca[k], cb[k]), k
    for c in (a, b, other):
        c.free()
