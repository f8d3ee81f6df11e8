"""The mapping criterion at the cell counts where its launch changes: one or two
cells a thread (an even number of cells in an array that starts on 16 bytes), and
eight, four, two or one row in flight.  Flags and reference index equal the
oracle's exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = (1, 2, 255, 131071, 131072, 131073, 262143, 262144, 524287, 524288, 524290)


def _field(mech, n, pattern, seed):
    """Cells on the mixing line: candidates (Z below 1e-4) at random, nowhere, in
    the last cell or in the first only."""
    g = np.random.default_rng(seed)
    Z = g.uniform(1e-3, 1.0, n)
    if pattern == "random":
        Z[g.uniform(size=n) < 0.5] = 5e-5
    elif pattern == "last":
        Z[-1] = 0.0
    elif pattern == "first":
        Z[0] = 0.0
    Y = np.outer(synth.stream_fuel(mech), Z) + np.outer(synth.stream_oxidiser(mech), 1.0 - Z)
    Y += 1e-12 * g.uniform(size=Y.shape)
    return g.uniform(300.0, 1500.0, n), Y


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("pattern", ["random", "none", "first", "last"])
def test_flags_and_reference_at_every_launch(pattern, offset):
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism("small")
    o, c = Oracle(mech), chem_for(mech)
    Yf, Yo = synth.stream_fuel(mech), synth.stream_oxidiser(mech)
    for n in SIZES:
        T, Y = _field(mech, n, pattern, 71 + n)
        buf = torch.zeros(Y.size + 1, dtype=torch.float64, device="cuda")
        buf[offset:offset + Y.size] = dev(Y).view(-1)
        Yd = buf[offset:offset + Y.size].view(Y.shape)
        assert Yd.data_ptr() % 16 == 8 * offset
        for use_T in (False, True):
            say("mapping", pattern, "offset", offset, n, use_T)
            flags, ref = c.map_reference(dev(T), dev(np.full(n, 1e6)), Yd, Yf, Yo, 1e-4, T_tol=300.0, use_T=use_T)
            want, wref = o.map_reference(T, Y, Yf, Yo, 1e-4, T_tol=300.0, use_T=use_T)
            assert int(ref.item()) == wref and np.array_equal(host(flags), want), (n, use_T)


def test_flags_of_a_53_species_field():
    """53 rows: whole groups of eight, four and two rows and the remainders."""
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism("mech53")
    o, c = Oracle(mech), chem_for(mech)
    Yf, Yo = synth.stream_fuel(mech), synth.stream_oxidiser(mech)
    for n in (1000, 131072, 262144, 524288):
        T, Y = _field(mech, n, "random", 91 + n)
        say("mapping mech53", n)
        flags, ref = c.map_reference(dev(T), dev(np.full(n, 1e6)), dev(Y), Yf, Yo, 1e-4)
        want, wref = o.map_reference(T, Y, Yf, Yo, 1e-4)
        assert int(ref.item()) == wref and np.array_equal(host(flags), want), n
