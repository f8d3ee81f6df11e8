"""The surrogate's network outside the range a trained network meets."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 100])
def test_gelu_of_an_overflow_is_infinite(n):
    """A pre-activation that overflows is infinite, and GELU(+inf) = +inf: with
    positive weights behind it every layer's result is +inf, and the outputs
    are infinite with the sign of their own weights."""
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism("mech53")
    dims, W = synth.SUR_DIMS, []
    for l in range(5):
        w = np.full((dims[l + 1], dims[l]), 1.0 / 256, np.float32)
        if l == 0:
            w[:] = 0.0
            w[:, 0] = 1e38          # times ln T = 6..8 (mean 0, spread 1 below)
        if l == 4:
            w[1::2] *= -1.0
        W += [w.ravel(), np.zeros(dims[l + 1], np.float32)]
    norm = np.zeros((6, 64), np.float32)
    norm[1] = norm[3] = 1.0
    c = chem_for(mech)
    c.surrogate_set_params(np.concatenate(W + [norm.ravel()]))
    f = synth.subsample(synth.field_mapped(400, seed=7), np.arange(n))
    args = dev(f.T), dev(f.p), dev(f.Y), dev(synth.surrogate_dt(n, 8))
    ref = np.broadcast_to(np.where(np.arange(64) % 2 == 0, np.inf, -np.inf), (n, 64))
    say("gelu of an overflow", n)
    assert np.array_equal(host(c.surrogate_forward(*args)), ref)
    assert np.array_equal(host(c.surrogate_forward_fused(*args)), ref)


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_forward_into_an_unaligned_array(offset):
    """The output array needs a float's alignment only: an array that starts 4, 8
    or 12 bytes past a 16-byte boundary receives the same values, and nothing
    around it is written."""
    from tests.gpu_util import chem_for, dev, say
    mech = synth.mechanism("mech53")
    n = 200                       # three full tiles of 64 rows and a ragged one
    c = chem_for(mech)
    c.surrogate_set_params(synth.surrogate_params(mech.n_species, seed=9))
    f = synth.subsample(synth.field_mapped(800, seed=10), np.arange(n))
    args = dev(f.T), dev(f.p), dev(f.Y), dev(synth.surrogate_dt(n, 11))
    say("surrogate forward, offset", offset)
    for forward in (c.surrogate_forward, c.surrogate_forward_fused):
        buf = torch.full((64 * n + 8,), 7.25, dtype=torch.float32, device="cuda")
        assert buf.data_ptr() % 16 == 0
        forward(*args, out=buf[offset:offset + 64 * n])
        assert torch.equal(buf[offset:offset + 64 * n].view(n, 64), forward(*args))
        assert (buf[:offset] == 7.25).all() and (buf[offset + 64 * n:] == 7.25).all()
