"""The per-cell kernel's branches against the oracle: the tabulated collision
integral over the whole temperature range (its ends and interval edges among
them) and the fit itself where the range is too wide for the table, a pure
species, rates with more than three factors a side, a reaction switched off
by an infinite ln A offset, and ragged block ends.

Bars: mu, lambda and D_s are sums of positive terms, a few hundred roundings
each, so 1e-12 per cell; the rates carry |ln K_c| ~ 100 times the rounding
and are differences, so 1e-12 of the row's largest."""
import copy

import numpy as np
import pytest
import torch

import synth
from conftest import normwise
from gpu_util import both, dev, gpu_cells, host
from paper_2202_02319_amd import htr

pytestmark = pytest.mark.gpu


def _case(ns, nr, N, eps=None, pure=False, high_order=False):
    mech = synth.make_mechanism(ns, nr, 7) if nr else synth.make_mechanism(max(ns, 3), 1, 7)
    if ns < mech.ns or eps is not None or high_order:
        mech = copy.deepcopy(mech)
    if ns < mech.ns:   # the first species, inert
        for k in ("W", "nasa7", "lj_sigma", "lj_epsk"):
            setattr(mech, k, getattr(mech, k)[:ns])
        mech.lnA = mech.beta = mech.Ea = np.zeros(0)
        mech.nu_f = mech.nu_r = np.zeros((0, ns), np.int32)
    if eps is not None:
        mech.lj_epsk = np.geomspace(*eps, mech.ns)
    if high_order:
        # both sides doubled where no coefficient passes the accepted 3
        k = np.where(np.maximum(mech.nu_f, mech.nu_r).max(axis=1) > 1, 1, 2)[:, None].astype(np.int32)
        assert (k > 1).any()
        mech.nu_f, mech.nu_r = mech.nu_f * k, mech.nu_r * k
        mech.lnA = mech.lnA - 12.0
    rng = np.random.default_rng(3)
    T = np.concatenate([np.geomspace(200.0, 6000.0, N - 12), 2.0 ** np.arange(8, 13), [200.0, 6000.0],
                        1000.0 * (1 + np.array([1, 2, -1, 8, 0]) * 2.0 ** -52)])
    T = np.clip(T, 200.0 * (1 + 1e-13), 6000.0 * (1 - 1e-13))
    Y = rng.dirichlet(np.ones(mech.ns), size=N).T
    if pure:
        Y[:] = 0.0
        Y[np.arange(N) % mech.ns, np.arange(N)] = 1.0
    g = synth.uniform_grid((N, 1, 1), 1e-4)
    return synth.Case("point", mech, g, np.ascontiguousarray(Y), T, np.full(N, 1.7e5), rng.standard_normal((3, N)) * 50)


@pytest.mark.parametrize("ns,nr,N,kw", [
    (2, 0, 300, {}), (3, 1, 257, {}), (9, 20, 511, {}), (12, 30, 300, {}), (1, 0, 100, {}),
    (5, 4, 300, dict(eps=(0.5, 5000.0))), (2, 0, 64, dict(eps=(120.0, 120.0))),
    (4, 2, 300, dict(pure=True)), (4, 2, 300, dict(pure=True, eps=(0.5, 5000.0))), (5, 3, 300, dict(high_order=True)),
])
def test_cells(ns, nr, N, kw):
    case = _case(ns, nr, N, **kw)
    o, g = both(case)
    U = o.prim_to_cons()
    ref, got = o.cells(U, case.T.copy()), gpu_cells(g, U, case.T.copy(), 0.0, None)
    assert np.abs(got[0] / ref[0] - 1).max() <= 1e-12
    for row in range(1, 5 + ns):
        assert np.abs(got[row] / ref[row] - 1).max() <= 1e-12, row
    assert normwise(got[5 + ns:6 + 2 * ns], ref[5 + ns:6 + 2 * ns]).max() <= 1e-12


def test_reaction_switched_off():
    case = synth.small_case(n=(20, 6, 1), seed=3, laser=False, mech=synth.case_c1().mech)
    less = copy.deepcopy(case)
    for k in ("lnA", "beta", "Ea", "nu_f", "nu_r"):
        setattr(less.mech, k, getattr(case.mech, k)[1:])
    out = []
    for c, d in ((case, [-np.inf, 0.0, 0.0, 0.0]), (less, [0.0] * 3)):
        _, g = both(c)
        U = htr.cons_from_case(g, c)
        z = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(3)]
        htr.htr_rk3_step(g, U, dev(c.T), z[0], z[1], 1, None, dev(d), g.new_work(), z[2])
        htr.htr_check(g)
        out.append((host(U), host(z[2])))
    assert normwise(out[0][0], out[1][0]).max() <= 1e-12
    assert normwise(out[0][1][None], out[1][1][None]).max() <= 1e-12
