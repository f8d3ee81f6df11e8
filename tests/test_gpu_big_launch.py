"""Entry points with one workgroup a cell, past the cell count at which that
exceeds a launch's 2^32 work-items: the workgroup integrator's evaluations, the
wavefront integrator's static schedule and single steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

KINDS = 5
CELLS = (1 << 23) + 3                # 512 threads a cell: 2^32 at 2^23 cells
WAVE_CELLS = (1 << 26) + 3           # 64 threads a cell


def _states(N, cells=CELLS):
    g = np.random.default_rng(29)
    T = torch.tensor(g.uniform(900.0, 2200.0, KINDS), device="cuda")
    Y = torch.tensor(np.ascontiguousarray(g.dirichlet(np.full(N, 0.5), KINDS).T), device="cuda")
    p = torch.full((cells,), 1.01325e6, dtype=torch.float64, device="cuda")
    kind = torch.arange(cells, device="cuda") % KINDS
    return T, Y, p, kind


def _all_like_the_first(out, n, first):
    out = out.view(-1, n)
    cells = out.shape[0]
    whole = cells // KINDS * KINDS
    assert (out[:whole].view(-1, KINDS, n) == first).all()
    assert (out[whole:] == first[:cells - whole]).all()


def test_rates_of_more_cells_than_one_launch_has_groups():
    """Every cell's rates equal those of the same state in a call of five."""
    from tests.gpu_util import chem_for, say
    N, n = 85, 86
    c = chem_for(synth.make_mechanism(N, 2 * N, 4, seed=61, name="launch86"))
    T, Y, p, kind = _states(N)
    first = torch.zeros(KINDS * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(T, p[:KINDS], Y, first)
    say("rates of", CELLS, "cells")
    f = torch.zeros(CELLS * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(T[kind].contiguous(), p, Y[:, kind].contiguous(), f)
    torch.cuda.synchronize()
    assert torch.isfinite(first).all() and first.view(KINDS, n)[:, 0].ne(0).all()
    _all_like_the_first(f, n, first.view(KINDS, n))


def test_steps_of_more_cells_than_one_launch_has_groups():
    """Every cell's fixed step equals that of the same state in a call of five."""
    from tests.gpu_util import chem_for, say
    N, n = 64, 65
    c = chem_for(synth.make_mechanism(N, 2 * N, 4, seed=62, name="launch65"))
    T, Y, p, kind = _states(N)
    y1, e1 = (torch.zeros(KINDS * n, dtype=torch.float64, device="cuda") for _ in range(2))
    c.rodas_step(T, p[:KINDS], Y, 1e-12, y1, e1)
    say("steps of", CELLS, "cells")
    yn, er = (torch.zeros(CELLS * n, dtype=torch.float64, device="cuda") for _ in range(2))
    c.rodas_step(T[kind].contiguous(), p, Y[:, kind].contiguous(), 1e-12, yn, er)
    torch.cuda.synchronize()
    assert torch.isfinite(y1).all() and torch.isfinite(e1).all()
    _all_like_the_first(yn, n, y1.view(KINDS, n))
    _all_like_the_first(er, n, e1.view(KINDS, n))


def test_static_schedule_of_more_cells_than_one_launch_has_groups():
    """Every cell is advanced, to the state of the same cell in a call of five."""
    from tests.gpu_util import chem_for, say
    mech = synth.mechanism("small")
    c = chem_for(mech, schedule=0, rtol=1e-2, atol=1e-4)   # one attempt a cell
    T, Y, p, kind = _states(mech.n_species, WAVE_CELLS)
    big_T, big_Y = T[kind].contiguous(), Y[:, kind].contiguous()
    T0 = T.clone()
    c.integrate(T, p[:KINDS], Y, 1e-12)
    say("static schedule,", WAVE_CELLS, "cells")
    status = torch.full((WAVE_CELLS,), 255, dtype=torch.uint8, device="cuda")
    c.integrate(big_T, p, big_Y, 1e-12, status=status)
    torch.cuda.synchronize()
    assert T.ne(T0).all() and (status == 0).all()
    _all_like_the_first(big_T, 1, T.view(KINDS, 1))
    for k in range(mech.n_species):
        _all_like_the_first(big_Y[k], 1, Y[k].view(KINDS, 1))


def test_wavefront_steps_of_more_cells_than_one_launch_has_groups():
    """Every cell's fixed step equals that of the same state in a call of five."""
    from tests.gpu_util import chem_for, say
    mech = synth.mechanism("small")
    n = mech.n_species + 1
    c = chem_for(mech)
    T, Y, p, kind = _states(mech.n_species, WAVE_CELLS)
    y1, e1 = (torch.zeros(KINDS * n, dtype=torch.float64, device="cuda") for _ in range(2))
    c.rodas_step(T, p[:KINDS], Y, 1e-12, y1, e1)
    say("steps of", WAVE_CELLS, "cells")
    yn, er = (torch.zeros(WAVE_CELLS * n, dtype=torch.float64, device="cuda") for _ in range(2))
    c.rodas_step(T[kind].contiguous(), p, Y[:, kind].contiguous(), 1e-12, yn, er)
    torch.cuda.synchronize()
    assert torch.isfinite(y1).all() and torch.isfinite(e1).all()
    _all_like_the_first(yn, n, y1.view(KINDS, n))
    _all_like_the_first(er, n, e1.view(KINDS, n))
