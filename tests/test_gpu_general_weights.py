"""Kernels that only meshes with general reconstruction weights reach: the tiled
edge pass (LDS tiles of 8, 16 and 32 edges) and the barotropic loops over weight
tables, with land, pentagons, FP32 and in batches.

Bounds: the oracle comparisons of the other kernel tests (1e-11 L2, 1e-10
largest, FP64; one loop 1e-12, and in FP32 12 substeps x 50 roundings x 6e-8
with a factor 10, 4e-4); forms of one kernel agree bit for bit.
"""
import numpy as np
import pytest

from oracle import ssprk_se as S
from oracle.layered import Setup
from synthetic import cases
from tests.parity_cases import vmix
from tests.test_gpu_factored_loop import _inputs
from tests.test_gpu_parity import _check_kernel, _noisy_state
from tests.test_gpu_split_pass import _with_general_weights
from tests.test_gpu_vmix import _assert_mix, _feuler_ref, _mix_errs

pytestmark = pytest.mark.gpu

CASES = {
    "hex12_L64": lambda: cases.c1(n=12, L=64, steps=1),
    "hex8_L100": lambda: cases.c1(n=8, L=100, steps=1),
    "sphere3_land_L7": lambda: cases.sphere_case(3, 7, 77, substeps=5, dt_btr=200.0),
    "sphere3_land_L8": lambda: cases.sphere_case(3, 8, 78, substeps=5, dt_btr=200.0),
}


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_13484_amd import ssprkse
    ssprkse.load()
    return ssprkse


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("variant", [-2, -1, 0, 1, 2])
def test_edge_pass_matches_the_oracle(dev, name, variant):
    case = _with_general_weights(CASES[name]())
    st_o = Setup.from_case(case)
    u, h = _noisy_state(case, steps=1)
    ubar, _ = S.split(u, h, st_o)
    zeta = S.ssh(h, st_o)
    ut1, G = S.baroclinic_feuler(u, u - ubar[:, None], zeta, h, case.params.dt, st_o)
    _, st = dev.state_from_case(case)
    if not st.try_edge_variant(variant):
        pytest.skip(f"variant {variant} does not fit: {dev.last_error()}")
    g_ut1, g_G = st.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)
    _check_kernel(f"feuler variant={variant} {name}, general weights", {"ut1": (g_ut1, ut1), "G": (g_G, G)})


@pytest.mark.parametrize("name", ["hex12_L64", "hex8_L100", "sphere3_land_L7"])
@pytest.mark.parametrize("variant", [-1, 0, 1, 2])
def test_edge_pass_with_mixing_matches_the_oracle(dev, name, variant):
    case = vmix(_with_general_weights(CASES[name]()))
    u, h, ubar, zeta, ut1, G = _feuler_ref(case)
    _, st = dev.state_from_case(case)
    if not st.try_edge_variant(variant):
        pytest.skip(f"variant {variant} does not fit: {dev.last_error()}")
    g_ut1, g_G = st.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)
    _assert_mix(f"feuler+mixing variant={variant} {name}, general weights", _mix_errs(g_ut1, g_G, ut1, G, ubar))


@pytest.mark.parametrize("mixing", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("make", [lambda: cases.c1(n=16, L=60, steps=3),
                                  lambda: cases.sphere_case(3, 9, 5, substeps=5, dt_btr=60.0)])
def test_edge_variants_agree(dev, make, precision, mixing):
    case = cases.with_params(_with_general_weights(make()), precision=precision)
    if mixing:
        case = vmix(case)
    out = {}
    for v in (-1, -2, 0, 1, 2):
        _, st = dev.state_from_case(case)
        if not st.try_edge_variant(v):
            assert v >= 0, dev.last_error()
            continue
        assert st.edge_variant == v
        assert st.step(3) == 0, dev.last_error()
        out[v] = st.read()
    assert len(out) > 2            # some tiled variant ran
    for v in out:
        for k in out[-1]:
            assert np.array_equal(out[-1][k], out[v][k]), (v, k)


LOOPS = {
    "one_patch_hex16": lambda: cases.c1(n=16, L=2, steps=1),
    "hex40": lambda: cases.c1(n=40, L=2, steps=1),
    "pentagons_sphere3": lambda: cases.sphere_case(3, 2, 5, substeps=5, dt_btr=100.0, land_fraction=0.0),
    "land_sphere4": lambda: cases.sphere_case(4, 2, 7, substeps=5, dt_btr=60.0),
}


@pytest.mark.parametrize("name", sorted(LOOPS))
@pytest.mark.parametrize("scheme", [2, 3])
@pytest.mark.parametrize("precision", [0, 1])
def test_loop_forms_agree_and_match_the_oracle(dev, name, scheme, precision):
    case = cases.with_params(_with_general_weights(LOOPS[name]()), precision=precision)
    inputs, dt = _inputs(case, 3), case.params.dt / case.params.substeps * 12
    out = {}
    for v in (0, 1, 2):
        _, st = dev.state_from_case(case)
        assert st.try_bt_variant(v), dev.last_error()
        out[v] = st.debug_barotropic_substep(scheme, 12, dt, *inputs)
    for v in (1, 2):
        for a, b in zip(out[0], out[v]):
            assert np.array_equal(a, b), v
    sub = S.barotropic_ssprk2_substep if scheme == 2 else S.barotropic_ssprk3_substep
    want = sub(*inputs, dt, 12, Setup.from_case(case))
    for a, b in zip(out[1], want):
        assert np.linalg.norm(a - b) <= (4e-4 if precision else 1e-12) * np.linalg.norm(b)


@pytest.mark.parametrize("precision", [0, 1])
def test_batch_of_general_and_factored_members_equals_alone(dev, precision):
    import torch
    stream = torch.cuda.Stream()
    cs = [cases.c1(n=24, L=5, substeps=12, dt_btr=10.0, steps=2), cases.sphere_case(4, 9, 5, substeps=11, dt_btr=60.0),
          cases.c1(n=12, L=66, substeps=7, dt_btr=10.0, steps=2), cases.sphere_case(3, 3, 6, substeps=4, dt_btr=60.0)]
    cs = [cases.with_params(_with_general_weights(c) if i % 2 == 0 else c, precision=precision, scheme=3) for i, c in enumerate(cs)]
    keep, b = [], dev.Batch(stream=stream)
    for c in cs:
        keep.append(dev.state_from_case(c, stream=stream))
        b.add(keep[-1][1])
    assert b.step(2) == 0
    for i, (c, (_, st)) in enumerate(zip(cs, keep)):
        _, alone = dev.state_from_case(c, stream=stream)
        assert alone.step(2) == 0
        got, want = st.read(), alone.read()
        for k in want:
            assert np.array_equal(got[k], want[k]), (i, k)
