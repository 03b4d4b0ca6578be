"""The curvilinear diffusive kernel's tiles against the oracle: 8 x 8 x 4 cells
on three active axes, 16 x 16 on two (whichever they are), 256 on one, each at
a whole number of tiles, one cell more and below one tile; odd and even
species counts, the largest among them.

Bar: each row is a difference of face fluxes that carry about a hundred
roundings, 1e2 x 1.1e-16 of the largest term, with one to two orders lost in
the differences: 1e-12 of the row's largest, as for the other right-hand
sides."""
import numpy as np
import pytest

import synth
from conftest import normwise
from gpu_util import both, gpu_rhs

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _case(n, ns, nr, flags=0):
    c = synth.small_case(n=n, ns=ns, nr=nr, seed=43, flags=flags)
    if sum(x > 1 for x in n) > 1:
        g = synth.wavy_grid(c.grid.n, c.grid.spacing(), amp=0.2, seed=7)
    else:
        g = synth.affine_grid(c.grid.n, c.grid.spacing(), np.diag([1.3 if x > 1 else 1.0 for x in n]))
    return synth.Case(c.name + "-curv", c.mech, g, c.Y, c.T, c.p, c.vel, flags=flags)


@pytest.mark.parametrize("n,ns,nr", [
    ((8, 8, 4), 5, 4), ((9, 17, 5), 4, 2), ((7, 3, 2), 3, 1), ((16, 8, 9), 12, 20), ((6, 9, 13), 9, 10),
    ((16, 32, 1), 5, 4), ((17, 1, 33), 6, 4), ((1, 15, 16), 5, 4), ((1, 1, 257), 4, 2), ((1, 40, 1), 3, 1),
    ((256, 1, 1), 5, 4),
])
def test_rhs(n, ns, nr):
    case = _case(n, ns, nr)
    o, g = both(case)
    U = o.prim_to_cons()
    ref = o.rhs(U, case.T.copy(), t=0.0)
    got, _ = gpu_rhs(g, U, case.T.copy(), 0.0, None)
    assert normwise(got, ref[0] if isinstance(ref, tuple) else ref).max() <= TOL
