"""What the host keeps between calls: batch tables of several chain sets, and
the pinned boxes that state reads go through (needs an MI355X)."""
import threading

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


def _chain(m, seed, p=None):
    return kcm.Chain(synth.sequence(m, seed), TYPES, p or params(kcm.KCM_MIXED), theta0=synth.random_dihedrals(m, seed))


# one atom workgroup, several, and a state that no longer fits a box (1 MiB)
@pytest.mark.parametrize("m", [1, 27, 1200, 2300])
def test_state_reads_agree_with_each_other(m):
    c = _chain(m, 70 + m)
    print(f"case=state-reads m={m}", flush=True)
    c.step(1)
    st = c.state()
    fp, fc = c.forces()
    assert np.array_equal(st["force"], fp + fc)
    assert np.array_equal(st["theta"], c.theta())
    # the links stay rigid: N-CA of every residue at its bond length
    x = st["xyz"].reshape(m, 10, 3)
    assert np.allclose(np.linalg.norm(x[:, 2] - x[:, 0], axis=1), 1.458, atol=1e-9)
    assert np.array_equal(np.abs(st["tau"]).max(), kcm.kcm_step([c], 0)[1][0].max_tau)
    c.free()


def test_reads_from_more_threads_than_boxes():
    chains = [_chain(20 + k, 80 + k) for k in range(6)]
    want = []
    for c in chains:
        c.step(2)
        want.append(c.state())
    got, errors = [None] * 6, []

    def read(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(50):
                    got[k] = chains[k].state()
                    for key in got[k]:
                        assert np.array_equal(got[k][key], want[k][key]), key
        except BaseException as e:  # reported by the test's thread
            errors.append(e)

    print("case=threads", flush=True)
    ts = [threading.Thread(target=read, args=(k,)) for k in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors


def test_more_chain_sets_in_turn_than_a_stream_keeps():
    # six sets in turn on one stream, short ones and one in nine launches,
    # with a set freed and another built in between
    p = params(kcm.KCM_MIXED)
    spec = [[5, 9], [30], [12, 12, 7], [200, 3], [26], [40, 2]]
    sets = [[_chain(m, 100 * k + i, p) for i, m in enumerate(ms)] for k, ms in enumerate(spec)]
    print("case=chain-sets", flush=True)
    for turn in range(3):
        for k in (0, 1, 2, 3, 4, 5, 1, 0):
            kcm.kcm_step(sets[k], 1 + turn)
        if turn == 0:
            for c in sets[2]:
                c.free()
            sets[2] = [_chain(m, 200 + i, p) for i, m in enumerate(spec[2])]
    its = [2 * (1 + 2 + 3), 2 * (1 + 2 + 3), 2 + 3, 6, 6, 6]
    for k, ms in enumerate(spec):
        for i, m in enumerate(ms):
            alone = _chain(m, 200 + i if k == 2 else 100 * k + i, p)
            kcm.kcm_step([alone], its[k])
            sa, sb = alone.state(), sets[k][i].state()
            for key in sa:
                assert np.array_equal(sa[key], sb[key]), (k, i, key)
            alone.free()
