"""Rates and Jacobian of any number of cells: how a call's cells are laid over
workgroups and wavefronts changes no result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

KINDS = 5
# one cell, one a CU and one more, two a CU, all wavefronts of a workgroup per CU
# (five for mech53, eight for small) and one more, several rounds
CELLS = (1, 3, 255, 256, 257, 512, 513, 1280, 1281, 2048, 2049, 5003)


@pytest.mark.parametrize("name", ["small", "mech53", "mech53pl", "mech63", "mech64"])
def test_every_cell_is_evaluated_alike(name):
    """Every cell's f and J equal, bit for bit, those of the same state in a call
    of five; those are compared with the oracle by the kernel tests."""
    from tests.gpu_util import chem_for, dev, say
    mech = synth.mechanism(name)
    N, n = mech.n_species, mech.n_species + 1
    g = np.random.default_rng(41)
    T, p = dev(g.uniform(900.0, 2200.0, KINDS)), dev(1.01325e6 * np.exp(g.uniform(-1.0, 1.0, KINDS)))
    Y = dev(np.ascontiguousarray(g.dirichlet(np.full(N, 0.5), KINDS).T))
    c = chem_for(mech)
    f1 = torch.zeros(KINDS, n, dtype=torch.float64, device="cuda")
    J1 = torch.zeros(KINDS, n, n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(T, p, Y, f1, J1)
    assert torch.isfinite(J1).all() and J1[:, 0].ne(0).any(dim=1).all()
    for cells in CELLS:
        kind = torch.arange(cells, device="cuda") % KINDS
        say("evaluation of", cells, "cells", name)
        f = torch.full((cells + 1, n), 7.25, dtype=torch.float64, device="cuda")
        J = torch.full((cells + 1, n, n), 7.25, dtype=torch.float64, device="cuda")
        c.eval_rhs_jac(T[kind].contiguous(), p[kind].contiguous(), Y[:, kind].contiguous(), f, J)
        assert torch.equal(f[:cells], f1[kind]) and torch.equal(J[:cells], J1[kind])
        assert (f[cells] == 7.25).all() and (J[cells] == 7.25).all()
