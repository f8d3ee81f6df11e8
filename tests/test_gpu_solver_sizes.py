"""Both integrators at the sizes where a register or panel layout begins or
ends: one fixed Rodas4 step and the right-hand side with its Jacobian against
the oracle, for seeded mechanisms of n = N + 1 unknowns.

n = 16, 24, 32, 40, 48 and 56 fill a padded wavefront matrix, 13, 17, 49 and 55
start the next size; 80, 81, 85 and 86 are whole panels of the workgroup kernel,
a last panel of one column, and the two sides of its evaluation's workgroup
sizes; 128 and 129 two and three rows a lane; at 136 and 138 the wavefronts
share fewer production-rate arrays, and 138 is the last size that fits.  (54, 64
and 65 unknowns are in the tests of the mechanisms of that size.)
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = (13, 16, 17, 24, 32, 40, 48, 49, 55, 56, 80, 81, 85, 86, 128, 129, 136, 138)


@pytest.mark.parametrize("n", SIZES)
def test_step_and_jacobian_match_oracle(n):
    """The step to 4 eps cond(M) on the scale of the state, the bound of the
    fixed-step tests: a solve with partial pivoting has a forward error of about
    cond(M) eps, once on each side, and the 4 covers the stage sums.  Rates and
    Jacobian within 20 of their rounding scale."""
    from tests.gpu_util import check_rhs_jac, chem_for, dev, host, say
    N, cells = n - 1, 6
    mech = synth.make_mechanism(N, 4 * N, 4, seed=40 + n, name=f"size{n}")
    g = np.random.default_rng(900 + n)
    T = g.uniform(900.0, 2200.0, cells)
    p = np.full(cells, 1.01325e6)
    Y = np.ascontiguousarray(g.dirichlet(np.full(N, 0.5), cells).T)
    field = synth.Field(T=T, p=p, Y=Y, dt=1e-6)
    o = Oracle(mech)
    c = chem_for(mech)
    say("sizes rhs_jac", n)
    f = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    J = torch.zeros(cells * n * n, dtype=torch.float64, device="cuda")
    c.eval_rhs_jac(dev(T), dev(p), dev(Y), f, J)
    torch.cuda.synchronize()
    check_rhs_jac(o, mech, field, host(f).reshape(cells, n), host(J).reshape(cells, n, n), f"n = {n}")
    hstep = 1e-9
    say("sizes rodas_step", n)
    yn = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    er = torch.zeros(cells * n, dtype=torch.float64, device="cuda")
    c.rodas_step(dev(T), dev(p), dev(Y), hstep, yn, er)
    torch.cuda.synchronize()
    yn, er = host(yn).reshape(cells, n), host(er).reshape(cells, n)
    for i in range(cells):
        y = np.concatenate([[T[i]], Y[:, i]])
        yo, eo, rc = o.rodas4_step(p[i], y, hstep)
        assert rc == 0
        if not np.all(np.isfinite(yo)):
            continue
        M = np.eye(n) / (0.25 * hstep) - o.jac(p[i], y)
        bound = max(1e-12, 4 * 2.2e-16 * np.linalg.cond(M))
        scale = np.abs(y) + np.abs(yo) + 1e-12
        assert np.max(np.abs(yn[i] - yo) / scale) <= bound
        assert np.max(np.abs(er[i] - eo) / scale) <= bound
