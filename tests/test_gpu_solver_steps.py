"""One fixed Rodas4 step of both integrators at the sizes where a register or
panel layout begins or ends, at steps for which the solution is well determined.

n = 16, 24, 32, 40, 48 and 56 fill a padded wavefront matrix, 13, 17, 49 and 55
start the next size; 65, 80 and 81 are a last panel of one column and of 16 in
the workgroup kernel; 128 and 129 two and three rows a lane; from 136 on the
wavefronts share production-rate arrays, and 138 is the last size that fits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = (13, 16, 17, 24, 32, 40, 48, 49, 55, 56, 65, 80, 81, 85, 86, 128, 129, 136, 138)
STEPS = 10.0 ** -np.arange(7.0, 23.0, 0.25)


def determined_step(o, p, y):
    """The longest step at which the oracle's is finite, cond(M) <= 1e6 and the
    tolerances are below 1e-8 of the scale; with its result and the tolerances.
    These are four times the oracle's own spread over eight runs with every entry
    of J moved by up to 1e-13 of its row's largest (the kernels' J is within
    5e-13, measured 6e-14) and the state by up to 4 eps, plus 64 eps of the scale
    for the stage sums."""
    n, J = y.size, o.jac(p, y)
    row = np.abs(J).max(axis=1)[:, None]
    for h in STEPS:
        cond = np.linalg.cond(np.eye(n) / (0.25 * h) - J)
        yo, eo, rc = o.rodas4_step(p, y, h)
        if cond > 1e6 or rc != 0 or not (np.isfinite(yo).all() and np.isfinite(eo).all()):
            continue
        g = np.random.default_rng(5)
        dy, de = np.zeros(n), np.zeros(n)
        for _ in range(8):
            Jp = J + 1e-13 * row * g.uniform(-1.0, 1.0, (n, n))
            yp = y * (1.0 + 4 * 2.0 ** -52 * g.uniform(-1.0, 1.0, n))
            y2, e2, _ = o.rodas4_step(p, yp, h, J=Jp)
            dy, de = np.maximum(dy, np.abs(y2 - yo)), np.maximum(de, np.abs(e2 - eo))
        scale = np.abs(y) + np.abs(yo) + 1e-12
        ty, te = 4 * dy + 64 * 2.0 ** -52 * scale, 4 * de + 64 * 2.0 ** -52 * scale
        if (ty / scale).max() < 1e-8 and (te / scale).max() < 1e-8:
            return h, cond, yo, eo, ty, te
    raise AssertionError("no such step")


@pytest.mark.parametrize("n", SIZES)
def test_determined_step_matches_oracle(n):
    from tests.gpu_util import chem_for, dev, host, say
    N, cells = n - 1, 6
    mech = synth.make_mechanism(N, 4 * N, 4, seed=40 + n, name=f"size{n}")
    g = np.random.default_rng(900 + n)
    T = g.uniform(900.0, 2200.0, cells)
    Y = np.ascontiguousarray(g.dirichlet(np.full(N, 0.5), cells).T)
    p = np.full(cells, 1.01325e6)
    o, c = Oracle(mech), chem_for(mech)
    say("determined steps", n)
    worst, hard = 0.0, 0
    for i in range(cells):
        y = np.r_[T[i], Y[:, i]]
        h, cond, yo, eo, ty, te = determined_step(o, p[i], y)
        hard += cond > 1e3
        yn = torch.zeros(n, dtype=torch.float64, device="cuda")
        er = torch.zeros(n, dtype=torch.float64, device="cuda")
        c.rodas_step(dev(T[i:i + 1]), dev(p[i:i + 1]), dev(Y[:, i:i + 1]), h, yn, er)
        torch.cuda.synchronize()
        worst = max(worst, (np.abs(host(yn) - yo) / ty).max(), (np.abs(host(er) - eo) / te).max())
    print(n, "worst / tolerance", worst, "cells with cond(M) > 1e3:", hard)
    assert hard >= cells // 2           # the elimination matters
    assert worst <= 1.0
