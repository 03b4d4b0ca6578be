"""The diffusive sweeps' tiles: three-dimensional grids of exactly one tile, one
cell more along each axis and axes of two and three cells (periodic images
inside a tile), even and odd species counts (the species go in twos), and an
ensemble whose members have one, two and three active axes, so that both
sweeps pass over each other's members.  Per RHS <= 1e-12 normwise against the
oracle; members bitwise equal to their single-grid runs."""
import numpy as np
import pytest
import torch

import synth
from conftest import normwise
from gpu_util import both, dev, gpu_rhs, host
from paper_2202_02319_amd import htr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nr", [(2, 0), (5, 4)])
@pytest.mark.parametrize("n", [(8, 8, 4), (9, 8, 4), (8, 9, 5), (2, 3, 2), (17, 3, 9), (3, 17, 5)])
def test_rhs(n, ns, nr):
    mech = synth.case_c1().mech if ns == 5 else synth.make_mechanism(2, 0, 3)
    case = synth.small_case(n=n, seed=9, mech=mech)
    case.laser.t0 = 0.0
    o, g = both(case)
    U = o.prim_to_cons()
    ref = o.rhs(U, case.T.copy(), t=2e-8)
    got, _ = gpu_rhs(g, U, case.T.copy(), 2e-8, case.laser)
    assert normwise(got, ref).max() <= 1e-12


def test_members_of_different_dimension():
    mech = synth.case_c1().mech
    cases = [synth.small_case(n=n, seed=10 + k, mech=mech) for k, n in
             enumerate([(9, 7, 6), (300, 1, 1), (17, 13, 1), (8, 8, 4), (1, 20, 3)])]
    ctx = htr.Context(mech, cases[0].grid)
    b = htr.Batch.from_cases(ctx, cases)
    U, T = htr.batch_state_from_cases(b, cases)
    t = torch.zeros(b.nmem, dtype=torch.float64, device="cuda")
    out = torch.empty_like(U)
    htr.htr_rhs_batched(b, U, T.clone(), t, out)
    htr.htr_batch_check(b)
    for m, c in enumerate(cases):
        _, g = both(c)
        single, _ = gpu_rhs(g, b.unpack(host(U), b.ctx.nv, m), c.T, 0.0, c.laser)
        assert np.array_equal(b.unpack(host(out), b.ctx.nv, m), single)
