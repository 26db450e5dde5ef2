"""Rounding of the implicit vertical mixing in mixed precision."""
import numpy as np
import pytest

from synthetic import cases
from tests.test_gpu_vmix import dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("L", [5, 30, 60, 100])
def test_the_solve_adds_no_more_rounding_than_the_stage(dev, mode, L):  # noqa: F811
    """Ten mixed-precision steps of a current of 0.3 m/s, against the same in
    FP64, with the mixing solved for and left out: the solve rounds relative to
    the change it makes, so the velocity's error grows by less than its own size
    (each stage rounds some tens of times without it, the solve once for the sum
    and in the change, which is small)."""
    case = cases.c1(n=24, L=L, steps=10)
    case.u[:] += 0.3 * np.cos(2 * np.pi * np.arange(len(case.u)) / len(case.u))[:, None]
    err = {}
    for mix in (0, 1):
        out = []
        for precision in (0, mode):
            c = cases.with_params(case, precision=precision, vmix=mix, nu_v=1.0e-4 if mix else 0.0, c_drag=1.0e-3 if mix else 0.0)
            _, st = dev.state_from_case(c)
            assert st.step(10) == 0, dev.last_error()
            out.append(st.read()["u"])
        err[mix] = np.linalg.norm(out[1] - out[0]) / np.linalg.norm(out[0])
    print(f"\n[column solve] mode {mode} L {L}: {err[0]:.2e} without, {err[1]:.2e} with mixing", flush=True)
    assert err[1] <= 2.0 * err[0]
