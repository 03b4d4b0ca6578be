"""Three-dimensional grids of few cells along an axis or two: the diffusive sweep
takes the tile shape of fewest tiles, so that no more blocks run than the 16 x 4 x 3
tiles would have (counted in the library's sources compiled for the CPU, whose
results are those of the oracle), and on the GPU each shape against the oracle at
1e-12 normwise, an ensemble of them bitwise the single grids."""
import numpy as np
import pytest
import torch

import cpu_build
import synth
from conftest import normwise
from gpu_util import both, gpu_rhs, host
from oracle import Oracle
from paper_2202_02319_amd import htr

#         8x8x4        8x4x8       4x8x8       16x4x3
SHAPES = [(17, 16, 4), (16, 4, 8), (4, 9, 16), (65, 2, 2), (33, 4, 3), (2, 3, 2), (9, 9, 9), (7, 2, 11)]


def _case(n):
    case = synth.small_case(n=n, seed=9, mech=synth.case_c1().mech)
    case.laser.t0 = 0.0
    return case


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return cpu_build.build(tmp_path_factory.mktemp("cpu"), [5])


@pytest.mark.parametrize("n", SHAPES)
def test_blocks_cpu(built, monkeypatch, n):
    lib = cpu_build.use(built, monkeypatch)
    case = _case(n)
    g = htr.Context.from_case(case)
    o = Oracle(case)
    U = torch.tensor(o.prim_to_cons())
    T, d = torch.tensor(case.T), torch.empty_like(U)
    lib.cpu_blocks(b"")
    htr.htr_rhs(g, U, T, 2e-8, case.laser, d)
    htr.htr_check(g)
    most = np.prod([-(-a // b) for a, b in zip(n, (16, 4, 3))])
    assert lib.cpu_blocks(b"k_diff") <= most
    assert normwise(d.numpy(), o.rhs(U.numpy(), case.T.copy(), t=2e-8)).max() <= 1e-12


@pytest.mark.parametrize("n,blocks", [((9, 17, 5), 10),     # 12, 10, 9 and 10 tiles: 4x8x8 not for a tenth
                                      ((4, 17, 17), 9),     # 15, 15, 9 and 30: but for more than a fifth
                                      ((10, 17, 9), 18)])   # 18, 20, 18 and 15: 16x4x3 not for less than a fifth
def test_weights_cpu(built, monkeypatch, n, blocks):
    lib = cpu_build.use(built, monkeypatch)
    case = _case(n)
    g = htr.Context.from_case(case)
    U = torch.tensor(Oracle(case).prim_to_cons())
    lib.cpu_blocks(b"")
    htr.htr_rhs(g, U, torch.tensor(case.T), 2e-8, case.laser, torch.empty_like(U))
    htr.htr_check(g)
    assert lib.cpu_blocks(b"k_diff") == blocks


@pytest.mark.gpu
@pytest.mark.parametrize("n", SHAPES)
def test_rhs(n):
    case = _case(n)
    o, g = both(case)
    U = o.prim_to_cons()
    got, _ = gpu_rhs(g, U, case.T.copy(), 2e-8, case.laser)
    assert normwise(got, o.rhs(U, case.T.copy(), t=2e-8)).max() <= 1e-12


@pytest.mark.gpu
def test_ensemble():
    cases = [_case(n) for n in SHAPES]
    ctx = htr.Context(cases[0].mech, cases[0].grid)
    b = htr.Batch.from_cases(ctx, cases)
    U, T = htr.batch_state_from_cases(b, cases)
    t = torch.full((b.nmem,), 2e-8, dtype=torch.float64, device="cuda")
    for grid in (0, 3):
        htr.htr_batch_set_tiling(b, -1, None, grid)
        out = torch.empty_like(U)
        htr.htr_rhs_batched(b, U, T.clone(), t, out)
        htr.htr_batch_check(b)
        for m, c in enumerate(cases):
            _, g = both(c)
            single, _ = gpu_rhs(g, b.unpack(host(U), b.ctx.nv, m), c.T, 2e-8, c.laser)
            assert np.array_equal(b.unpack(host(out), b.ctx.nv, m), single)
