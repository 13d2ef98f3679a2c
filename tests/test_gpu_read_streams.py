"""A state read on another stream than the chain's work waits for that work
where the streams are blocking ones, and reads work with either default of
pinned memory (needs an MI355X)."""
import ctypes as C
import os
import re
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from gpu_common import TYPES, params  # noqa: E402
from paper_1712_05012_amd import kcm  # noqa: E402

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def hip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    kcm.load_library()
    # the runtime that is loaded already
    path = re.search(r"/\S*libamdhip64\.so\S*", open("/proc/self/maps").read()).group(0)
    return C.CDLL(path)


def _stream(hip):
    s = C.c_void_p()
    assert hip.hipStreamCreate(C.byref(s)) == 0  # a blocking stream
    return s.value


# the reads of each size: one kernel into pinned memory, and the copies of a state too large for it
@pytest.mark.parametrize("m,n_iter", [(15, 2000), (2300, 40)])
@pytest.mark.parametrize("reader", ["another", "null"])
def test_read_on_another_stream_sees_the_queued_steps(hip, m, n_iter, reader):
    work, other = _stream(hip), _stream(hip)
    seq, th = synth.sequence(m, 60), synth.random_dihedrals(m, 60)
    a, b = (kcm.Chain(seq, TYPES, params(kcm.KCM_MIXED), theta0=th) for _ in range(2))
    print(f"case=read-streams m={m} reader={reader}", flush=True)
    torch.cuda.synchronize()
    kcm.kcm_step([a], n_iter)
    want = a.state()
    kcm.kcm_step([b], n_iter, stream=work, report=False)
    got = kcm.kcm_get_state(b.handle, stream=other if reader == "another" else 0)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert np.array_equal(kcm.kcm_get_state(b.handle, stream=work)["theta"], want["theta"])
    for s in (work, other):
        assert hip.hipStreamSynchronize(C.c_void_p(s)) == 0 and hip.hipStreamDestroy(C.c_void_p(s)) == 0
    a.free()
    b.free()


def test_a_call_without_iterations_moves_no_work_to_its_stream(hip):
    work, other = _stream(hip), _stream(hip)
    seq, th = synth.sequence(15, 62), synth.random_dihedrals(15, 62)
    a, b = (kcm.Chain(seq, TYPES, params(kcm.KCM_MIXED), theta0=th) for _ in range(2))
    print("case=read-streams no iterations", flush=True)
    torch.cuda.synchronize()
    kcm.kcm_step([a], 2000)
    want = a.state()
    kcm.kcm_step([b], 2000, stream=work, report=False)
    kcm.kcm_step([b], 0, stream=other, report=False)
    got = kcm.kcm_get_state(b.handle, stream=other)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    for s in (work, other):
        assert hip.hipStreamSynchronize(C.c_void_p(s)) == 0 and hip.hipStreamDestroy(C.c_void_p(s)) == 0
    a.free()
    b.free()


def test_reads_do_not_depend_on_the_default_of_pinned_memory():
    # the records and the boxes are polled: coherent memory, also where the
    # environment makes pinned memory non-coherent unless asked otherwise
    code = """
import sys
sys.path[:0] = [%r, %r]
import torch
import numpy as np
from gpu_common import TYPES, params
import synth
from paper_1712_05012_amd import kcm
c = kcm.Chain(synth.sequence(30, 61), TYPES, params(kcm.KCM_MIXED), theta0=synth.random_dihedrals(30, 61))
for k in range(20):
    rep = c.step(1)
    st = c.state()
    f = c.forces()
    assert rep.iterations == k + 1 and np.abs(st["tau"]).max() == rep.max_tau
    assert np.array_equal(st["force"], f[0] + f[1]) and np.array_equal(st["theta"], c.theta())
c.free()
print("reads agree")
""" % (ROOT, HERE)
    for value in ("0", "1"):
        r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, HIP_HOST_COHERENT=value), timeout=100,
                           capture_output=True, text=True)
        print(f"case=pinned-default HIP_HOST_COHERENT={value} rc={r.returncode}", flush=True)
        assert r.returncode == 0 and "reads agree" in r.stdout, r.stderr[-2000:]
