"""Large mechanisms whose Gibbs energies exceed the range of exp: the reverse
rates come from differences of logarithms, so only the differences matter.

Adding the same heat to every atom of a kind (a6_k += shift, per atom) changes no
reaction, as every reaction is balanced, but carries |g / RT| of the larger
species to 700-2300 at 200-600 K (oxides and fluorocarbons reach it at 300 K),
where exp(+-g) is infinite or zero."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


def _shifted(name, shift):
    m = copy.deepcopy(synth.mechanism(name))
    m.nasa[:, 5] += shift * m.composition.sum(axis=1)
    return m


@pytest.mark.parametrize("name", ["mech64", "mech64pl", "mech130"])
@pytest.mark.parametrize("shift", [-4e4, 4e4])
def test_reverse_rates_at_large_gibbs_energies(name, shift):
    """Rates, Jacobian and a fixed step against the oracle, within the bounds of
    the other kernel tests (20 rounding scales, 5e-13 of a row, 4 eps cond(M))
    times (64 + 5 G) / 64: those take the terms of the exponents to be up to
    64, here five energies of up to G = max |g / RT| enter each."""
    from tests.gpu_util import chem_for, dev, host, rounding_scale, say
    mech = _shifted(name, shift)
    N, n = mech.n_species, mech.n_species + 1
    T = np.array([210.0, 300.0, 300.0, 600.0])
    cells, hstep = T.size, 1e-12
    p = np.full(cells, 1.01325e6)
    Y = np.ascontiguousarray(np.random.default_rng(23).dirichlet(np.full(N, 0.5), cells).T)
    o, c = Oracle(mech), chem_for(mech)
    say("large Gibbs energies", name, shift)
    f = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    J = torch.zeros(cells * n * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(dev(T), dev(p), dev(Y), f, J)
    yn = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    er = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    c.rodas_step(dev(T), dev(p), dev(Y), hstep, yn, er)
    torch.cuda.synchronize()
    f, J = host(f).reshape(cells, n), host(J).reshape(cells, n, n)
    yn, er = host(yn).reshape(cells, n), host(er).reshape(cells, n)
    assert np.isfinite(f).all() and np.isfinite(J).all() and np.isfinite(yn).all()
    for i in range(cells):
        y = np.r_[T[i], Y[:, i]]
        _, h, s = o.thermo(T[i])
        G = np.abs(h - s).max()
        assert G > 700.0
        more = (64.0 + 5.0 * G) / 64.0
        fo, Jo = o.rhs(p[i], y), o.jac_cs(p[i], y)
        sc = rounding_scale(o, mech, T[i], p[i], Y[:, i]) * more
        assert np.all(np.abs(f[i] - fo) <= 20.0 * sc)
        dJ = np.abs(J[i] - Jo)
        assert np.all(dJ[:, 1:] * np.abs(y[1:])[None, :] <= 20.0 * sc[:, None])
        rows = np.abs(Jo).max(axis=1)
        assert np.all(dJ.max(axis=1) <= 5e-13 * more * rows)
        yo, eo, rc = o.rodas4_step(p[i], y, hstep)
        assert rc == 0 and np.isfinite(yo).all()
        bound = max(1e-12, 4 * 2.2e-16 * np.linalg.cond(np.eye(n) / (0.25 * hstep) - o.jac(p[i], y))) * more
        assert bound < 1e-6
        scale = np.abs(y) + np.abs(yo) + 1e-12
        assert np.max(np.abs(yn[i] - yo) / scale) <= bound
        assert np.max(np.abs(er[i] - eo) / scale) <= bound
