"""Temperatures below zero: the rates have no value there (ln T), and none may
come back.  A stage of a failing attempt can come to such a temperature; its
rates must make the attempt non-finite, so that it is rejected, in the wavefront
integrator (up to 64 unknowns) and in the workgroup integrator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

MECHS = ("small", "mech53", "mech53pl", "mech63", "mech64", "mech64pl")


@pytest.mark.parametrize("name", MECHS)
def test_rates_jacobian_and_step_have_no_value_below_zero(name):
    """Wherever the oracle's rates are not finite (all but the species in no
    reaction), the kernels' rates and rows of the Jacobian are not either, and
    no component of a fixed step is."""
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism(name)
    N, n = mech.n_species, mech.n_species + 1
    T = np.array([-50.0, -0.5, -1e-3, -300.0, -2500.0])
    cells = T.size
    p = np.full(cells, 1.01325e6)
    Y = np.ascontiguousarray(np.random.default_rng(17).dirichlet(np.full(N, 0.5), cells).T)
    o, c = Oracle(mech), chem_for(mech)
    say("rates below 0 K", name)
    f = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    J = torch.zeros(cells * n * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(dev(T), dev(p), dev(Y), f, J)
    yn = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    er = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    c.rodas_step(dev(T), dev(p), dev(Y), 1e-9, yn, er)
    torch.cuda.synchronize()
    f, J = host(f).reshape(cells, n), host(J).reshape(cells, n, n)
    for i in range(cells):
        y = np.r_[T[i], Y[:, i]]
        none = ~np.isfinite(o.rhs(p[i], y))
        assert none[0] and none.sum() >= n - 2
        assert not np.isfinite(f[i][none]).any()
        assert not np.isfinite(J[i][none]).any()
    assert not np.isfinite(host(yn)).any() and not np.isfinite(host(er)).any()


@pytest.mark.parametrize("name,cells", [("small", 4000), ("mech53", 300), ("mech64", 300)])
def test_step_with_a_stage_below_zero_has_no_value(name, cells):
    """Steps much too long for the state: where one of the oracle's stages is
    below 0 K its step is not finite, and neither is the kernel's."""
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism(name)
    n = mech.n_species + 1
    f = synth.field_small(cells, seed=19) if name == "small" else synth.field_bimodal(name, cells, 19, shuffle=True)
    o, c = Oracle(mech), chem_for(mech)
    bad = 0
    for h in (1e-7, 1e-5, 1e-3):
        say("stages below 0 K", name, cells, h)
        yn = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
        er = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
        c.rodas_step(dev(f.T), dev(f.p), dev(f.Y), h, yn, er)
        torch.cuda.synchronize()
        got = np.isfinite(host(yn).reshape(cells, n)).all(axis=1)
        ref = np.array([np.isfinite(o.rodas4_step(f.p[i], np.r_[f.T[i], f.Y[:, i]], h)[0]).all()
                        for i in range(cells)])
        print(name, h, "not finite:", (~ref).sum(), "by the oracle,", (~got).sum(), "on the GPU")
        assert not got[~ref].any()
        bad += (~ref).sum()
    assert bad >= cells // 100


def test_no_cell_is_carried_on_below_zero():
    """At a tolerance so loose that an attempt can end below 0 K, such a state is
    accepted only as a call's last step (its rates are not looked at any more);
    before that the cell ends with a status.  The oracle has at most two such
    cells in 20000."""
    from tests.gpu_util import chem_for, run_integrate, say
    mech = synth.mechanism("small")
    for seed in (101, 102, 103):
        f = synth.field_small(20000, seed=seed)
        T, _, _, st, _, _ = Oracle(mech).integrate_batch(f.T, f.p, f.Y, 1e-3, rtol=0.1, atol=1e-2, max_steps=5000)
        ref = int(((T <= 0.0) & (st == 0)).sum())
        say("loose tolerance", seed)
        c = chem_for(mech, rtol=0.1, atol=1e-2, max_steps=5000)
        out = run_integrate(c, f, dt=1e-3)
        got = int(((out["T"] <= 0.0) & (out["status"] == 0)).sum())
        print("below 0 K with status 0: oracle", ref, "GPU", got)
        assert ref <= 2 and got <= 2
