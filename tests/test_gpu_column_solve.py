"""The column solve of the implicit vertical mixing at the layer counts where
its rounds change: none, the DPP round alone, the first shuffled round, below,
at and above 32 and 64 layers (the wrapped round, the last lane, two register
chunks), and the most layers.  Bounds are those of the mixing parity tests;
FP32 against FP64 input stays within 128 roundings of 6e-8 times the largest
pivot ratio of these columns (below 10): 1e-4.
"""
import pytest

from synthetic import cases
from tests.helpers import rel_l2
from tests.parity_cases import vmix
from tests.test_gpu_vmix import _assert_mix, _feuler_ref, _mix_errs, dev  # noqa: F401

pytestmark = pytest.mark.gpu

LAYERS = [1, 2, 3, 4, 5, 8, 9, 17, 31, 32, 33, 48, 63, 64, 65, 66, 127, 128]


@pytest.mark.parametrize("L", LAYERS)
def test_column_solve_at_any_layer_count(dev, L):  # noqa: F811
    case = vmix(cases.c1(n=8, L=L, steps=1))
    u, h, ubar, zeta, ut1, G = _feuler_ref(case)
    _, st = dev.state_from_case(case)
    g_ut1, g_G = st.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)
    _assert_mix(f"column solve L={L}", _mix_errs(g_ut1, g_G, ut1, G, ubar))
    _, st = dev.state_from_case(cases.with_params(case, precision=1))
    g_ut1, _ = st.debug_baroclinic_feuler(u, ubar, zeta, h, case.params.dt)
    assert rel_l2(g_ut1 + ubar[:, None], ut1 + ubar[:, None]) <= 1e-4
