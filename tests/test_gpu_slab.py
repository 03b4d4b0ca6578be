"""The boundary kernel's dense order of the cells next to non-periodic
boundaries: the smallest bounded axes (eight nodes: the layers of both sides
and two cells between), every axis bounded, cell counts around a block's 64.
Per RHS <= 1e-12 normwise against the oracle, the bar of the boundary tests."""
import pytest

import synth
from conftest import normwise
from gpu_util import both, gpu_rhs
from test_gpu_boundaries import _case

pytestmark = pytest.mark.gpu

W, I, O = synth.BC_WALL, synth.BC_INFLOW, synth.BC_OUTFLOW


@pytest.mark.parametrize("n,bc,flags", [
    ((8, 8, 8), ((I, O), (W, W), (O, O)), 0),
    ((9, 8, 11), ((O, O), (W, W), (W, W)), synth.FORCE_TENO),
    ((8, 1, 1), ((O, O), (0, 0), (0, 0)), 0),
    ((70, 1, 1), ((W, O), (0, 0), (0, 0)), synth.FORCE_TENO),
    ((8, 10, 1), ((I, O), (O, O), (0, 0)), 0),
    ((5, 6, 33), ((0, 0), (0, 0), (W, O)), synth.VISC_OFF),
    ((64, 3, 8), ((0, 0), (0, 0), (O, W)), 0),
])
def test_rhs(n, bc, flags):
    case = _case(n, bc, flags)
    o, g = both(case)
    U = o.prim_to_cons()
    ref, hrr_o = o.rhs(U, case.T.copy(), t=2e-8, want_hrr=True)
    got, _, hrr_g = gpu_rhs(g, U, case.T.copy(), 2e-8, case.laser, want_hrr=True)
    assert normwise(got, ref).max() <= 1e-12
    assert normwise(hrr_g[None], hrr_o[None]).max() <= 1e-12
