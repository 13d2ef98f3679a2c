"""The cell list that k_chain builds by matching keys inside each wave (chains of
at most 256 atoms) is a stable sort by cell (needs an MI355X).
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


# one to four waves with full and partial last ones; extended chains with many
# cells (several to a thread of the scan) and compact ones with many atoms to a
# cell; large cells put a whole chain into one
@pytest.mark.parametrize("cell_size", [0.0, 2.0, 60.0])
@pytest.mark.parametrize("fold", ["coil", "extended"])
@pytest.mark.parametrize("m", [1, 6, 7, 12, 13, 19, 20, 25])
def test_cells_are_a_stable_sort(m, fold, cell_size):
    th = synth.random_dihedrals(m, 90 + m) if fold == "coil" else np.full(2 * m, np.pi * 0.98)
    p = params(kcm.KCM_FP64, **({"cell_size": cell_size} if cell_size else {}))
    c = kcm.Chain(synth.sequence(m, 90 + m), TYPES, p, theta0=th)
    print(f"case=cell-match m={m} fold={fold} cell={cell_size}", flush=True)
    kcm.kcm_step([c], 1, check=False)
    cells, xyz = c.cells(), c.state()["xyz"]
    order, start, dims = np.asarray(cells["order"]), np.asarray(cells["cell_start"]), np.asarray(cells["dims"])
    assert len(start) == np.prod(dims) + 1 and start[0] == 0 and start[-1] == 10 * m
    assert np.array_equal(np.sort(order), np.arange(10 * m))
    u = (xyz - cells["origin"]) / cells["cell"]
    key = np.clip(np.floor(u).astype(int), 0, dims - 1)
    key = (key[:, 2] * dims[1] + key[:, 1]) * dims[0] + key[:, 0]
    # an atom within rounding of a cell's border may lie on either side
    sure = np.abs(u - np.rint(u)).min(axis=1) > 1e-9
    of_slot = np.repeat(np.arange(len(start) - 1), np.diff(start))
    assert np.array_equal(key[order][sure[order]], of_slot[sure[order]])
    for b, e in zip(start[:-1], start[1:]):
        assert np.all(np.diff(order[b:e]) > 0)
    c.free()
