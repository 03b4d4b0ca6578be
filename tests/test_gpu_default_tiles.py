"""The default tile shape by the grid's size: each of the four shapes where its
rule picks it, and the right-hand side bitwise that of 16x4x4 tiles (every face
is evaluated once with the same arithmetic whatever the tile)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, host
from paper_2202_02319_amd import htr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shape", [
    ((32, 16, 16), (16, 4, 4)), ((12, 12, 12), (16, 4, 4)), ((24, 24, 24), (8, 8, 4)), ((83, 13, 9), (8, 8, 4)),
    ((83, 61, 5), (8, 8, 4)), ((8, 12, 16), (8, 4, 8)), ((4, 15, 16), (4, 8, 8)),
])
def test_default_shape(n, shape):
    case = synth.small_case(n=n, seed=47, ns=5, nr=4, T_base=1500.0, mech=synth.case_c1().mech)
    out = []
    for set_16 in (False, True):
        g = htr.Context.from_case(case)
        if set_16:
            htr.htr_set_tiling(g, (16, 4, 4), 0)
        else:
            assert htr.htr_get_tiling(g) == (shape, 0)
        U = htr.cons_from_case(g, case)
        d = torch.empty_like(U)
        htr.htr_rhs(g, U, dev(case.T), 0.0, None, d, None)
        htr.htr_check(g)
        out.append(host(d))
    assert np.array_equal(out[0], out[1])
