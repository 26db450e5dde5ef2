"""Resident barotropic loops beside other work on the device.

The workgroups of a resident loop wait for each other, and other streams can
keep some of them off the device for as long as the others wait.  Such a loop
is called off and done patch by patch instead; results are the same bits.
"""
import numpy as np
import pytest

from synthetic import cases
from tests.test_gpu_factored_loop import MESHES, _inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_13484_amd import ssprkse
    ssprkse.load()
    return ssprkse


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("scheme,M", [(2, 1), (3, 2), (3, 21), (2, 12)])
@pytest.mark.parametrize("precision", [0, 1])
def test_called_off_loop_gives_the_same_bits(dev, name, scheme, M, precision):
    """Host arrays, and device arrays in the caller's numbering; the next loops
    of the same state, admitted and called off in turn, too."""
    import torch
    case = cases.with_params(MESHES[name](), precision=precision)
    inputs, dt = _inputs(case, 3), case.params.dt / case.params.substeps * M
    _, ref = dev.state_from_case(case)
    assert ref.try_bt_variant(1)
    want = ref.debug_barotropic_substep(scheme, M, dt, *inputs)
    _, st = dev.state_from_case(case)
    assert st.try_bt_variant(2), dev.last_error()
    for off in (True, False, True, True, False):
        st.call_off_loops(off)
        got = st.debug_barotropic_substep(scheme, M, dt, *inputs)
        ins = [torch.from_numpy(a).cuda() for a in inputs]
        outs = [torch.full_like(t, 5.0) for t in ins]
        st.barotropic_substep_noalloc(scheme, M, dt, *ins, *outs)
        torch.cuda.synchronize()
        for a, b, c in zip(want, got, outs):
            assert np.array_equal(a, b), off
            assert np.array_equal(a, c.cpu().numpy()), off


@pytest.mark.parametrize("name", ["two_patches_hex20", "hex64", "land_sphere5"])
@pytest.mark.parametrize("scheme,precision", [(2, 0), (3, 0), (3, 1)])
def test_device_arrays_after_a_wait_that_ran_out(dev, name, scheme, precision):
    """The loop on device arrays, whose error word no host call reads: a wait
    that runs out (forced with a one-poll limit) costs a second pass and leaves
    nothing behind for the next call of this or another state."""
    import torch
    case = cases.with_params(MESHES[name](), precision=precision)
    inputs, dt = _inputs(case, 9), case.params.dt / case.params.substeps * 15
    _, ref = dev.state_from_case(case)
    assert ref.try_bt_variant(1)
    want = ref.debug_barotropic_substep(scheme, 15, dt, *inputs)
    _, st = dev.state_from_case(case)
    _, other = dev.state_from_case(case)
    assert st.try_bt_variant(2) and other.try_bt_variant(2), dev.last_error()
    ins = [torch.from_numpy(a).cuda() for a in inputs]
    for state, spins in ((st, 1), (st, 1), (other, 0), (st, 0), (st, 1), (other, 0)):
        state.set_barrier_spins(spins)
        outs = [torch.full_like(t, 5.0) for t in ins]
        state.barotropic_substep_noalloc(scheme, 15, dt, *ins, *outs)
        torch.cuda.synchronize()
        for a, b in zip(want, outs):
            assert np.array_equal(a, b.cpu().numpy()), spins


@pytest.mark.parametrize("precision", [0, 1])
def test_called_off_batch_equals_alone(dev, precision):
    import torch
    stream = torch.cuda.Stream()
    specs = [(24, 5, 12), (12, 66, 25), (40, 3, 17), (16, 9, 2), (20, 2, 1)]
    cs = [cases.with_params(cases.c1(n=n, L=L, substeps=M, dt_btr=10.0, member=i, steps=2), precision=precision)
          for i, (n, L, M) in enumerate(specs)]
    keep, b = [], dev.Batch(stream=stream)
    for c in cs:
        keep.append(dev.state_from_case(c, stream=stream))
        b.add(keep[-1][1])
    for off in (True, False, True):
        keep[0][1].call_off_loops(off)
        assert b.step(1) == 0
    for c, (_, st) in zip(cs, keep):
        _, alone = dev.state_from_case(c, stream=stream)
        assert alone.try_bt_variant(1)
        assert alone.step(3) == 0
        got, want = st.read(), alone.read()
        for k in want:
            assert np.array_equal(got[k], want[k]), k


def test_loops_that_fill_the_device_on_several_streams(dev):
    """Batches and single states whose loops each need most of an empty device,
    stepped together on streams of their own, with their column kernels and a
    large copy between the loops: no wait runs out and every state has the bits
    it reaches alone with a launch per substep."""
    import torch
    specs = [(352, 1, True), (288, 0, True), (340, 1, False), (290, 0, False)]   # cells a side, precision, batch
    runs = []
    for i, (n, precision, batch) in enumerate(specs):
        case = cases.with_params(cases.c1(n=n, L=3, substeps=12, dt_btr=5.0, member=i, steps=2), precision=precision)
        stream = torch.cuda.Stream()
        _, st = keep = dev.state_from_case(case, stream=stream)
        run = st
        if batch:
            run = dev.Batch(stream=stream)
            run.add(st)
            run.compile()
            assert run.launches_per_step() < 50       # one launch per loop, or it would be 36 more
        runs.append((case, keep, run))
    a = torch.empty(1 << 27, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    side = torch.cuda.Stream()
    for _ in range(8):
        for _, _, run in runs:
            run.step_async(2)
        with torch.cuda.stream(side):
            b.copy_(a)
    torch.cuda.synchronize()
    for case, (_, st), run in runs:
        assert run.sync() == 0, dev.last_error()
        _, alone = dev.state_from_case(case)
        assert alone.try_bt_variant(1)
        assert alone.step(16) == 0
        got, want = st.read(), alone.read()
        for k in want:
            assert np.array_equal(got[k], want[k]), k


def test_state_created_while_its_stream_is_captured(dev):
    """Creation is recorded, not run: the counters of its loops are clear once
    the state is initialised, and replays between steps do no harm."""
    import torch
    case = cases.c1(n=48, L=3, substeps=12, dt_btr=5.0, steps=1)
    stream = torch.cuda.Stream()
    dm, ref = dev.state_from_case(case, stream=stream)
    assert ref.bt_variant == 2 and ref.step(3) == 0
    want = ref.read()
    x, g = torch.zeros(1, device="cuda"), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        x += 1
        st = dev.DeviceState(dm, case.params, stream=stream)
    st.buf.fill_(255)                       # memory that held something else before
    torch.cuda.synchronize()
    st.init(case.h, case.u, case.rho, case.h_ref)
    for _ in range(3):
        assert st.step(1) == 0
        with torch.cuda.stream(stream):
            g.replay()
        torch.cuda.synchronize()
    got = st.read()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert x.item() == 3


def test_state_created_after_an_error_of_the_callers(dev):
    """An error that the caller's own runtime call left behind is not taken for
    one of the state's creation."""
    import ctypes
    import torch
    case = cases.c1(n=24, L=2, substeps=12, dt_btr=5.0, steps=1)
    dm = dev.DeviceMesh(case.mesh, case.H, case.cell_mask)
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    value = ctypes.c_int()
    assert hip.hipDeviceGetAttribute(ctypes.byref(value), -5, 0) != 0     # no such attribute
    st = dev.DeviceState(dm, case.params)
    hip.hipGetLastError()
    st.init(case.h, case.u, case.rho, case.h_ref)
    assert st.step(1) == 0
    torch.cuda.synchronize()
