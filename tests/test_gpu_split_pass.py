"""The forward-Euler pass split by cells (factored reconstruction weights) and
the direct pass it replaces, which meshes with any other weights keep.

FP64: each within 1e-11 (relative L2) of the oracle, the bound of the other
per-kernel comparisons.  FP32: a term of the tendency rounds some tens of times
(6e-8 each), so the two passes agree to 1e-5 of the tendency's size.
"""
from dataclasses import replace

import numpy as np
import pytest

from oracle import ssprk_se as S
from oracle.layered import Setup
from synthetic import cases

pytestmark = pytest.mark.gpu

OPTIONS = {"plain": {}, "vmix": {"vmix": 1}, "del4": {"hdiff": 1, "nu_h": 1.0e12}, "iso": {"vcoord": 1}}


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_13484_amd import ssprkse
    ssprkse.load()
    return ssprkse


def _with_general_weights(case):
    """Some weight pairs scaled by 1 + 1e-9: no longer of the factored form."""
    w, eoe = case.mesh.weightsOnEdge.copy(), case.mesh.edgesOnEdge
    w[(eoe + np.arange(len(eoe))[:, None]) % 7 == 0] *= 1 + 1e-9
    return replace(case, mesh=replace(case.mesh, weightsOnEdge=w))


def _fields(case, seed=8):
    rng = np.random.default_rng(seed)
    st = Setup.from_case(case)
    u = np.where(st.edge_mask[:, None], rng.normal(0, 0.2, case.u.shape), 0.0)
    h = np.where(st.cell_mask[:, None], case.h * (1 + 1e-3 * rng.random(case.h.shape)), case.h)
    ubar, _ = S.split(u, h, st)
    return st, u, ubar, S.ssh(h, st), h


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("option", sorted(OPTIONS))
@pytest.mark.parametrize("make,L", [("hex", 1), ("hex", 63), ("hex", 64), ("hex", 65), ("sphere", 2), ("sphere", 128)])
def test_pass_matches_the_oracle(dev, make, L, option, general):
    if make == "hex":
        case = cases.c1(n=10, L=L, steps=1)
    else:
        case = cases.sphere_case(2, L, 4, substeps=5, dt_btr=60.0)
    kw = dict(OPTIONS[option])
    if make == "sphere" and "nu_h" in kw:
        kw["nu_h"] = 1.0e15
    case = cases.with_params(case, **kw)
    if general:
        case = _with_general_weights(case)
    st, u, ubar, zeta, h = _fields(case)
    want_u, want_G = S.bfe(u, u - ubar[:, None], ubar, zeta, h, case.params.dt, st)
    _, ds = dev.state_from_case(case)
    got_u, got_G = ds.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)
    scale = np.linalg.norm(want_u + ubar[:, None])   # ut1 = u1 - ubar may be small against u1
    assert np.linalg.norm(got_u - want_u) <= 1e-11 * scale
    assert np.linalg.norm(got_G - want_G) <= 1e-11 * np.linalg.norm(want_G)


@pytest.mark.parametrize("L", [20, 100])
def test_fp32_passes_agree(dev, L):
    case = cases.with_params(cases.sphere_case(3, L, 4, substeps=5, dt_btr=60.0), precision=1)
    _, u, ubar, zeta, h = _fields(case)
    out = []
    for c in (case, _with_general_weights(case)):
        _, ds = dev.state_from_case(c)
        out.append(ds.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)[0])
    tendency = np.linalg.norm(out[0] - (u - ubar[:, None]))
    assert np.linalg.norm(out[0] - out[1]) <= 1e-5 * tendency + 1e-6 * np.linalg.norm(u)


def test_steps_of_both_passes_stay_together(dev):
    """Whole steps, also through the stages that add the barotropic velocity."""
    case = cases.with_params(cases.sphere_case(3, 9, 4, substeps=6, dt_btr=60.0), scheme=3)
    out = []
    for c in (case, _with_general_weights(case)):
        _, ds = dev.state_from_case(c)
        assert ds.step(2) == 0
        out.append(ds.read())
    # the scaled weights themselves move the flow by up to 1e-9 of it
    for k in ("u", "h", "ubar"):
        assert np.linalg.norm(out[0][k] - out[1][k]) <= 1e-8 * np.linalg.norm(out[0][k]), k
