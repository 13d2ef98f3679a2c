"""What the autotuner times, with the device calls replaced: the graph depth is
a setting only of calls in nine launches, and every depth runs the same number
of iterations."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from paper_1712_05012_amd import autotune, kcm  # noqa: E402


class _Chain:
    def __init__(self, seq, types, p, theta0=None, stream=None):
        self.n_atoms = 10 * len(seq)

    def cells(self, stream):
        return {"cell": 4.4}

    def free(self):
        pass


def _runs(monkeypatch, sizes, depths):
    """(shape, depth set, iterations) of every timed kcm_step, and the tuner's result."""
    now = {"shape": 0, "depth": 1}
    steps = []
    monkeypatch.setattr(kcm, "Chain", _Chain)
    monkeypatch.setattr(kcm, "kcm_set_force_variant", lambda v: now.update(shape=v))
    monkeypatch.setattr(kcm, "kcm_set_graphs", lambda d: now.update(depth=d))
    monkeypatch.setattr(kcm, "kcm_step", lambda c, n, stream=None, report=True: steps.append((now["shape"], now["depth"], n)))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    items = [(synth.sequence(m, m), synth.random_dihedrals(m, m)) for m in sizes]
    res = autotune.tune(synth.residue_types(), items, kcm.KCM_MIXED, cell_sizes=(0.0, 3.6), variants=(0, 2),
                        depths=depths, iters=2, warmup=1)
    return steps[1::2], res  # each timed run follows a warm-up


def test_two_launch_sets_are_timed_once_for_all_depths(monkeypatch):
    sizes = (12, 30, 21)
    assert kcm.kcm_iteration_launches(sizes) == 2
    runs, res = _runs(monkeypatch, sizes, (1, 4, 8))
    assert [r[0] for r in runs] == [0, 2, 0, 2]  # edges times shapes
    # the table lists every depth, with one measurement, and the pick is the first
    assert len(res.table) == 12 and res.graph_depth == 1
    for k in range(0, 12, 3):
        assert len({r for *_, r in res.table[k:k + 3]}) == 1


def test_depths_of_nine_launch_sets_run_the_same_iterations(monkeypatch):
    sizes = (12, 300)
    assert kcm.kcm_iteration_launches(sizes) == 9
    runs, res = _runs(monkeypatch, sizes, (1, 4, 8))
    assert [r[1] for r in runs] == [1, 4, 8] * 4
    assert {r[2] for r in runs} == {16}
    assert len(res.table) == 12 and np.isfinite(res.atom_steps_per_s)
