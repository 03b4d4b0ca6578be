"""Mechanisms without a table of the collision integral (a range of T* of more than
ten octaves; a single species) on every route of the per-cell kernel: persistent
grids and ensembles bitwise the one-block-per-256-cells result, with as many
blocks as were asked for, and curvilinear grids against the oracle (per RHS
<= 1e-12 normwise, the bar of the curvilinear tests)."""
import copy

import numpy as np
import pytest
import torch

import cpu_build
import synth
from conftest import normwise
from gpu_util import both, dev, gpu_rhs, host
from oracle import Oracle
from paper_2202_02319_amd import htr


def _mech(ns):
    if ns == 1:
        return synth.single_species(0.02897)
    mech = copy.deepcopy(synth.case_c1().mech if ns == 5 else synth.make_mechanism(ns, 20, 7))
    mech.lj_epsk = np.geomspace(0.5, 5000.0, ns)
    return mech


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return cpu_build.build(tmp_path_factory.mktemp("cpu"), [1, 5])


@pytest.mark.parametrize("ns,table", [(1, False), (5, False), (5, True)])
def test_persistent_blocks_cpu(built, monkeypatch, ns, table):
    lib = cpu_build.use(built, monkeypatch)
    mech = synth.case_c1().mech if table else _mech(ns)
    case = synth.small_case(n=(40, 33, 1), seed=3, mech=mech, laser=False)
    g = htr.Context.from_case(case)
    U = torch.tensor(Oracle(case).prim_to_cons())
    out = []
    for grid in (0, 1, 2):
        htr.htr_set_tiling(g, None, grid)
        T, d = torch.tensor(case.T), torch.empty_like(U)
        lib.cpu_largest_grid()
        htr.htr_rhs(g, U, T, 0.0, None, d)
        htr.htr_check(g)
        blocks = lib.cpu_largest_grid()
        assert blocks == grid if grid else blocks > 2
        out.append((d, T))
    for d, T in out[1:]:
        assert np.array_equal(d, out[0][0]) and np.array_equal(T, out[0][1])


@pytest.mark.gpu
@pytest.mark.parametrize("ns", [1, 5, 9])
def test_persistent_grid_and_ensemble(ns):
    mech = _mech(ns)
    cases = [synth.small_case(n=n, seed=20 + k, mech=mech) for k, n in enumerate([(21, 9, 7), (33, 20, 1)])]
    single = []
    for c in cases:
        g = htr.Context.from_case(c)
        U = htr.cons_from_case(g, c)
        for grid in (0, 1, 3):
            htr.htr_set_tiling(g, None, grid)
            T, d = dev(c.T), torch.empty_like(U)
            htr.htr_rhs(g, U, T, 0.0, c.laser, d)
            htr.htr_check(g)
            if grid == 0:
                single.append((host(d), host(T)))
            else:
                assert np.array_equal(host(d), single[-1][0]) and np.array_equal(host(T), single[-1][1])
    ctx = htr.Context(mech, cases[0].grid)
    b = htr.Batch.from_cases(ctx, cases)
    for grid in (0, 2):
        htr.htr_batch_set_tiling(b, -1, None, grid)
        U, T = htr.batch_state_from_cases(b, cases)
        t = torch.zeros(b.nmem, dtype=torch.float64, device="cuda")
        d = torch.empty_like(U)
        htr.htr_rhs_batched(b, U, T, t, d)
        htr.htr_batch_check(b)
        for m in range(b.nmem):
            assert np.array_equal(b.unpack(host(d), ctx.nv, m), single[m][0])


@pytest.mark.gpu
@pytest.mark.parametrize("n,ns", [((13, 7, 6), 5), ((17, 11, 1), 9), ((9, 8, 5), 1)])
def test_curvilinear(n, ns):
    c = synth.small_case(n=n, seed=21, mech=_mech(ns))
    grid = synth.wavy_grid(c.grid.n, c.grid.spacing(), amp=0.25, seed=7)
    case = synth.Case("wide-wavy", c.mech, grid, c.Y, c.T, c.p, c.vel, laser=c.laser)
    o, g = both(case)
    U = o.prim_to_cons()
    ref = o.rhs(U, case.T.copy(), t=2e-8)
    got, _ = gpu_rhs(g, U, case.T.copy(), 2e-8, case.laser)
    assert normwise(got, ref).max() <= 1e-12
