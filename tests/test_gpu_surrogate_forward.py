"""Raw network outputs of both inference launches against the oracle's network.

chem_surrogate_forward and chem_surrogate_forward_fused run one kernel in two
instantiations: every row of a call written to the caller's rows, and listed rows
of a chunk written transposed, as the acceptance kernel reads them.  Comparing
them with each other says little, so each is compared with the oracle's
bfloat16 emulation (FP64 sums, the same roundings), every row, at sizes around a
tile of 64 rows; and across the first one's chunk of 2^24 rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2011_07978_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = (1, 17, 63, 64, 65, 128, 129, 700)
CHUNK = 1 << 24


def _params(N, seed):
    return synth.surrogate_params(N, seed=seed, weight_scale=1.5, out_sd=(1.0, 1.0),
                                  out_bias=synth.surrogate_increment_bias(N, seed + 1, 1e-7, 0.2))


@pytest.mark.parametrize("name", ["small", "mech53"])
@pytest.mark.parametrize("entry", ["surrogate_forward", "surrogate_forward_fused"])
def test_every_row_matches_the_emulation(name, entry):
    """Largest error 5e-3 of the largest output (an activation that rounds to the
    other bfloat16 neighbour), half of all outputs within 1e-7 of it (FP32
    against FP64 sums), and on average a quarter of what bfloat16 itself does,
    the bounds of the forward test at one size; padded outputs are zero."""
    from tests.gpu_util import chem_for, dev, host, say
    mech = synth.mechanism(name)
    N = mech.n_species
    P = _params(N, 51)
    c = chem_for(mech)
    c.surrogate_set_params(P)
    err, effect, scale = [], [], 0.0
    for n in SIZES:
        f = (synth.field_small(n, seed=52 + n) if name == "small"
             else synth.subsample(synth.field_mapped(4 * n + 40, seed=52 + n), np.arange(n)))
        dt = synth.surrogate_dt(n, 53 + n)
        X = np.stack([oracle.mlp_features(N, f.T[i], f.p[i], f.Y[:, i], dt[i]) for i in range(n)])
        emu = oracle.mlp_forward(P, X, N + 3, bf16_emulation=True)[:, :N + 1]
        exact = oracle.mlp_forward(P, X, N + 3, bf16_emulation=False)[:, :N + 1]
        say(entry, name, n)
        got = host(getattr(c, entry)(dev(f.T), dev(f.p), dev(f.Y), dev(dt)))
        assert got.shape == (n, 64) and np.all(got[:, N + 1:] == 0.0)
        e, s = np.abs(got[:, :N + 1] - emu), np.abs(emu).max()
        assert e.max() <= 5e-3 * s, n
        err.append(e.ravel())
        effect.append(np.abs(exact - emu).ravel())
        scale = max(scale, s)
    err, effect = np.concatenate(err), np.concatenate(effect)
    print(entry, name, "median", np.median(err) / scale, "mean", err.mean(), "bf16 effect", effect.mean())
    assert np.median(err) <= 1e-7 * scale
    assert err.mean() < 0.25 * effect.mean()


def test_forward_past_its_chunk():
    """Rows on both sides of 2^24 and of the ragged end equal those of the same
    states in a call of seven."""
    from tests.gpu_util import chem_for, dev, say
    mech = synth.mechanism("small")
    kinds, n = 7, CHUNK + 100
    c = chem_for(mech)
    c.surrogate_set_params(_params(mech.n_species, 61))
    f = synth.field_small(kinds, seed=62)
    T, p, Y, d = dev(f.T), dev(f.p), dev(f.Y), dev(synth.surrogate_dt(kinds, 63))
    first = c.surrogate_forward(T, p, Y, d)
    kind = torch.arange(n, device="cuda") % kinds
    say("surrogate forward", n, "rows")
    out = c.surrogate_forward(T[kind].contiguous(), p[kind].contiguous(), Y[:, kind].contiguous(), d[kind].contiguous())
    whole = n // kinds * kinds
    assert (out[:whole].view(-1, kinds, 64) == first).all()
    assert (out[whole:] == first[:n - whole]).all()


def test_narrow_and_wide_tiles_agree():
    """Calls of up to 4096 rows run in tiles of 16 rows, larger ones in tiles of
    64: the same bits for every row, at ragged ends too."""
    from tests.gpu_util import chem_for, dev, say
    mech = synth.mechanism("mech53")
    c = chem_for(mech)
    c.surrogate_set_params(_params(mech.n_species, 71))
    f = synth.subsample(synth.field_mapped(20000, seed=72), np.arange(5003))
    dt = synth.surrogate_dt(5003, 73)

    def forward(lo, hi):
        return c.surrogate_forward(dev(f.T[lo:hi]), dev(f.p[lo:hi]), dev(f.Y[:, lo:hi]), dev(dt[lo:hi]))

    say("tile widths")
    narrow = torch.cat([forward(0, 1), forward(1, 16), forward(16, 33), forward(33, 4096), forward(4096, 5003)])
    for n in (4095, 4096, 4097, 4160, 5003):
        assert torch.equal(forward(0, n), narrow[:n]), n
