"""State read-out: what was set comes back in the caller's order, bit for bit,
for read-outs of one pinned slot and of many, with and without renumbering."""
import numpy as np
import pytest

from synthetic import cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_13484_amd import ssprkse
    ssprkse.load()
    return ssprkse


@pytest.mark.parametrize("name,make", [
    ("hex8, one layer", lambda L: cases.c1(n=8, L=L, steps=1)),                                    # a few kB
    ("sphere4", lambda L: cases.sphere_case(4, L, 5, substeps=5, dt_btr=60.0)),                    # renumbered
    ("sphere6", lambda L: cases.sphere_case(6, L, 5, substeps=5, dt_btr=60.0, land_fraction=0.0)),  # many slots
    ("hex200", lambda L: cases.c1(n=200, L=L, steps=1)),                                           # many, as numbered
])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("L", [1, 41])
def test_read_returns_what_was_set(dev, name, make, precision, L):
    case = cases.with_params(make(L), precision=precision, tracer=1)
    rng = np.random.default_rng(1)
    c, sea = case.mesh.cellsOnEdge, case.cell_mask.astype(bool)
    wet = sea[c[:, 0]] & sea[c[:, 1]]
    u = np.where(wet[:, None], rng.normal(0, 0.1, case.u.shape), 0.0)
    h = case.h * (1 + 1e-4 * rng.random(case.h.shape))
    T = np.where(sea[:, None], rng.normal(10, 1, case.h.shape), 0.0)
    dm = dev.DeviceMesh(case.mesh, case.H, case.cell_mask)
    st = dev.DeviceState(dm, case.params)
    st.init(h, u, case.rho, case.h_ref)
    st.set_tracer(T)
    for _ in range(2):
        got = st.read()
        assert np.array_equal(got["h"], h)
        assert np.array_equal(got["u"], u if precision == 0 else u.astype(np.float32).astype(np.float64))
        assert np.array_equal(st.read_tracer(), T)
        assert np.allclose(got["zeta"], np.where(sea, h.sum(1) - case.H, 0.0), rtol=0, atol=1e-9)
        he = 0.5 * (h[c[:, 0]] + h[c[:, 1]])
        want = np.where(wet, (he * got["u"]).sum(1) / np.where(wet, he.sum(1), 1.0), 0.0)
        assert np.allclose(got["ubar"], want, rtol=0, atol=1e-12)


@pytest.mark.parametrize("make", [lambda: cases.c1(n=40, L=7, steps=1),                                    # as numbered
                                  lambda: cases.sphere_case(5, 41, 5, substeps=5, dt_btr=60.0)])           # renumbered
@pytest.mark.parametrize("precision", [0, 1])
def test_read_without_pinned_memory(dev, make, precision):
    """Where no pinned host memory is to be had the state still reads, the same."""
    case = cases.with_params(make(), precision=precision, tracer=1)
    dm = dev.DeviceMesh(case.mesh, case.H, case.cell_mask)
    st = dev.DeviceState(dm, case.params)
    st.init(case.h, case.u, case.rho, case.h_ref)
    st.set_tracer(np.where(case.cell_mask.astype(bool)[:, None], case.rho * 0.01, 0.0))
    assert st.step(2) == 0
    want, T = st.read(), st.read_tracer()
    st.plain_reads()
    got = st.read()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert np.array_equal(st.read_tracer(), T)


def test_read_from_a_thread_on_another_device(dev):
    """A state reads whatever device is current, and leaves it current."""
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("one device")
    case = cases.c1(n=40, L=7, steps=1)
    with torch.cuda.device(0):
        _, st = dev.state_from_case(case, device="cuda:0", stream=torch.cuda.Stream())
        want = st.read()
    with torch.cuda.device(1):
        got = st.read()
        assert torch.cuda.current_device() == 1
    for k in want:
        assert np.array_equal(got[k], want[k]), k


def test_read_of_nothing_waits_for_the_steps(dev):
    import torch
    case = cases.c1(n=128, L=40, steps=1)
    stream = torch.cuda.Stream()
    _, st = dev.state_from_case(case, stream=stream)
    st.step_async(60)
    assert dev.load().sse_read_state(st.handle, None, None, None, None) == dev.SSE_OK
    assert stream.query()


_CLOSE_IN_CAPTURE = """
import threading
import torch
from paper_2105_13484_amd import ssprkse as dev
from synthetic import cases
for other_thread in (False, True):
    stream = torch.cuda.Stream()
    dm, st = dev.state_from_case(cases.c1(n=24, L=7, steps=1), stream=stream)
    st.read()
    x, g = torch.zeros(1, device="cuda"), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()

    def close():
        st.close()
        dm.close()

    with torch.cuda.graph(g, stream=stream):
        x += 1
        if other_thread:
            t = threading.Thread(target=close)
            t.start()
            t.join()
        else:
            close()
        x += 1
    g.replay()
    torch.cuda.synchronize()
    assert x.item() == 2
print("captured")
"""


def test_last_state_and_mesh_closed_while_a_graph_is_captured(dev):
    """The pool's pinned memory goes with the last state and mesh of a process
    (hence a process of its own); a graph that is being captured meanwhile is not broken."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", _CLOSE_IN_CAPTURE], cwd=root, capture_output=True, text=True, timeout=100)
    assert res.returncode == 0 and "captured" in res.stdout, res.stderr
