"""The convective sweep's launches, counted in the library's sources compiled for
the CPU: with central faces forced the lean kernel runs alone, on few tiles too;
where few tiles may hold TENO faces, their variables are dealt to several blocks
of the full kernel, and where too many for that, the lean kernel goes first.
Results as the oracle's (1e-12 normwise)."""
import pytest
import torch

import cpu_build
import synth
from conftest import normwise
from oracle import Oracle
from paper_2202_02319_amd import htr


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return cpu_build.build(tmp_path_factory.mktemp("cpu"), [5])


CENTRAL = synth.FORCE_CENTRAL | synth.CHEM_OFF
#                       grid, flags, blocks of the lean and of the full kernel
@pytest.mark.parametrize("n,flags,lean,full", [
    ((40, 1, 1), CENTRAL, 9, 0),                        # 1 tile, a variable a block
    ((17, 17, 1), CENTRAL, 4 * 9, 0),                   # 16 x 16 tiles
    ((17, 17, 1), synth.CHEM_OFF, 0, 4 * 9),
    ((17, 3185, 1), CENTRAL | synth.VISC_OFF, 400, 0),  # no second run
    ((17, 3185, 1), synth.CHEM_OFF | synth.VISC_OFF, 400, 400),
])
def test_launches(built, monkeypatch, n, flags, lean, full):
    lib = cpu_build.use(built, monkeypatch)
    case = synth.small_case(n=n, seed=6, mech=synth.case_c1().mech, flags=flags, laser=False)
    g = htr.Context.from_case(case)
    o = Oracle(case)
    U = torch.tensor(o.prim_to_cons())
    T, d = torch.tensor(case.T), torch.empty_like(U)
    for name, blocks in ((b"k_conv_lean", lean), (b"6k_convI", full)):
        lib.cpu_blocks(b"")
        htr.htr_rhs(g, U, T.clone(), 0.0, None, d)
        htr.htr_check(g)
        assert lib.cpu_blocks(name) == blocks
    assert normwise(d.numpy(), o.rhs(U.numpy(), case.T.copy())).max() <= 1e-12
