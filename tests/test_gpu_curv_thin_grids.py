"""The curvilinear diffusive kernel's tiles on thin grids: on three axes the shape
of fewest tiles, and along the one long axis of a grid of at most four cells along
the others the longest tile that a block can stage.  Blocks counted in the
library's sources compiled for the CPU; results against the oracle at 1e-12
normwise, the bar of the other tiles."""
import pytest
import torch

import cpu_build
import synth
from conftest import normwise
from gpu_util import both, gpu_rhs
from oracle import Oracle
from paper_2202_02319_amd import htr

#         grid, tiles
SHAPES = [((62, 2, 2), 2), ((2, 32, 2), 2), ((2, 3, 43), 3), ((4, 4, 28), 2), ((3, 19, 3), 1), ((4, 4, 14), 1),
          ((65, 2, 1), 2), ((1, 4, 63), 1), ((9, 4, 17), 6), ((2, 9, 8), 2), ((8, 8, 4), 1), ((9, 17, 5), 10),
          ((3, 2, 2), 1)]


def _case(n):
    c = synth.small_case(n=n, ns=5, nr=4, seed=43, laser=False)
    return synth.Case(c.name, c.mech, synth.wavy_grid(n, c.grid.spacing(), amp=0.2, seed=7), c.Y, c.T, c.p, c.vel)


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return cpu_build.build(tmp_path_factory.mktemp("cpu"), [5])


@pytest.mark.parametrize("n,tiles", SHAPES)
def test_blocks_cpu(built, monkeypatch, n, tiles):
    lib = cpu_build.use(built, monkeypatch)
    case = _case(n)
    g = htr.Context.from_case(case)
    o = Oracle(case)
    U = torch.tensor(o.prim_to_cons())
    T, d = torch.tensor(case.T), torch.empty_like(U)
    lib.cpu_blocks(b"")
    htr.htr_rhs(g, U, T, 0.0, None, d)
    htr.htr_check(g)
    assert lib.cpu_blocks(b"k_curv_diff") == tiles
    ref = o.rhs(U.numpy(), case.T.copy(), t=0.0)
    assert normwise(d.numpy(), ref).max() <= 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("n", [n for n, _ in SHAPES])
def test_rhs(n):
    case = _case(n)
    o, g = both(case)
    U = o.prim_to_cons()
    got, _ = gpu_rhs(g, U, case.T.copy(), 0.0, None)
    assert normwise(got, o.rhs(U, case.T.copy(), t=0.0)).max() <= 1e-12
