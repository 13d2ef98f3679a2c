"""Atoms with more candidates than one set of the force kernel's start bits maps
(2,048), in both instances of the kernel, against the oracle (needs an MI355X).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import DTHETA_TOL, F_TOL, TAU_TOL, build_pair, compare_step, params  # noqa: E402
from paper_1712_05012_amd import kcm  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kcm.load_library()


# the cutoff covers all, or nearly all, of a coil of 2,150 or 4,400 atoms: one
# set of start bits and a part, and three sets
@pytest.mark.parametrize("m,cutoff", [(215, 200.0), (440, 90.0)])
@pytest.mark.parametrize("terms", [kcm.KCM_TERM_ELEC | kcm.KCM_TERM_VDW, kcm.KCM_TERM_ALL])
@pytest.mark.parametrize("precision", [kcm.KCM_FP64, kcm.KCM_MIXED])
def test_more_candidates_than_one_set_of_start_bits(precision, terms, m, cutoff):
    p = params(precision, cutoff=cutoff, terms=terms)
    gpu, ref, th = build_pair(m, 11 + m, p)
    print(f"case=many-candidates precision={precision} terms={terms} m={m}", flush=True)
    st, o, err = compare_step(gpu, ref, th, p)
    d = np.linalg.norm(o["r"] - o["r"].mean(axis=0), axis=1)
    assert (np.linalg.norm(o["r"] - o["r"][np.argmin(d)], axis=1) < cutoff).sum() > 2048
    assert err["status"] == 0 and err["F"] <= F_TOL
    assert err["tau"] <= TAU_TOL[precision] and err["dtheta"] <= DTHETA_TOL[precision]
    gpu.free()
