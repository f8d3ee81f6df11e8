"""Rates, Jacobian and steps on both sides of 200 K.  The wavefront integrator
keeps the species factors of the reverse rates as logarithms below it and as
exponentials from it on; the workgroup integrator uses logarithms throughout.
Every mechanism here has reactions that miss a second reactant, a second and a
third product, so the sentinels of missing slots count in both forms."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

TEMPERATURES = (60.0, 120.0, 199.9, 200.0, 200.1, 230.0)


@pytest.mark.parametrize("name", ["small", "mech53", "mech53pl", "mech63", "mech64", "mech64pl"])
def test_rates_and_jacobian_across_200_K(name):
    """Against the oracle within the bounds of the other kernel tests (20
    rounding scales; 5e-13 of a row), times (64 + 5 G) / 64: those take the
    terms of the exponents to be up to 64, here five energies of up to G =
    max |g / RT| enter each.  The static and the queue schedule read the records
    from different places, so one short advance of both is compared bit for
    bit."""
    from tests.gpu_util import chem_for, dev, host, rounding_scale, run_integrate, say
    mech = synth.mechanism(name)
    assert (mech.reactants[:, 1] < 0).any() and (mech.products[:, 1] < 0).any() and (mech.products[:, 2] < 0).any()
    N, n = mech.n_species, mech.n_species + 1
    T = np.repeat(TEMPERATURES, 2)
    cells = T.size
    p = np.full(cells, 1.01325e6)
    Y = np.ascontiguousarray(np.random.default_rng(37).dirichlet(np.full(N, 0.5), cells).T)
    o, c = Oracle(mech), chem_for(mech)
    say("rates across 200 K", name)
    f = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    J = torch.zeros(cells * n * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(dev(T), dev(p), dev(Y), f, J)
    torch.cuda.synchronize()
    f, J = host(f).reshape(cells, n), host(J).reshape(cells, n, n)
    worst = [0.0, 0.0, 0.0]
    for i in range(cells):
        y = np.r_[T[i], Y[:, i]]
        _, h, s = o.thermo(T[i])
        more = (64.0 + 5.0 * np.abs(h - s).max()) / 64.0
        fo, Jo = o.rhs(p[i], y), o.jac_cs(p[i], y)
        assert np.isfinite(fo).all() and np.isfinite(Jo).all()
        sc = rounding_scale(o, mech, T[i], p[i], Y[:, i]) * more
        live = sc > 0                      # species in some reaction
        assert np.all(f[i][~live] == 0.0) and np.all(J[i][~live] == 0.0)
        worst[0] = max(worst[0], (np.abs(f[i] - fo)[live] / sc[live]).max())
        dJ = np.abs(J[i] - Jo)
        worst[1] = max(worst[1], (dJ[live, 1:] * np.abs(y[1:])[None, :] / sc[live, None]).max())
        rows = np.abs(Jo).max(axis=1)
        worst[2] = max(worst[2], (dJ.max(axis=1)[live] / (rows[live] * more)).max())
    print(name, "worst f, J by column, J by row:", worst)
    assert worst[0] <= 20.0 and worst[1] <= 20.0 and worst[2] <= 5e-13
    field = synth.Field(T=T, p=p, Y=Y, dt=1e-12)
    a, b = run_integrate(c, field, schedule=0), run_integrate(c, field, schedule=1)
    assert np.array_equal(a["T"], b["T"]) and np.array_equal(a["Y"], b["Y"])
    assert (a["status"] == 0).all() and np.isfinite(a["Y"]).all()
