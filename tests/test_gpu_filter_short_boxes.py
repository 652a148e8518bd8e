"""Filter passes whose halo in one launch is longer than the box, so that its
cells wrap around the box more than once."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,tile,passes", [
    (1, (2,), (2,), 16),                # two launches of eight passes: a halo of four boxes
    (1, (6,), (2,), 15),                # halos of eight and seven cells on six
    (2, (2, 40), (2, 20), 8),           # halos of four on two cells
    (2, (48, 2), (12, 2), 7),
    (3, (2, 8, 2), (2, 4, 2), 4),       # halos of two on two cells
    (3, (2, 2, 2), (2, 2, 2), 3),
])
def test_halo_longer_than_the_box(D, n, tile, passes, prec):
    """Bound as for any pass: it rounds a sum of at most 3^D terms of weight 1
    in all (the weights are powers of two)."""
    from paper_1906_06306_amd.sim import PicSim
    sim = PicSim(synth.small_random(D, n, 2, seed=7, field_amp=0.05), tile=tile, precision=prec)
    rng = np.random.default_rng(passes)
    _, _, Jv = sim.field_views()
    Jv.copy_(torch.as_tensor(rng.standard_normal(tuple(Jv.shape)), device=Jv.device))
    ref = Jv.double().cpu().numpy().reshape(3, -1).copy()
    scale = np.abs(ref).max()
    sim.filter_current(passes)
    _, _, J = sim.fields_host(0)
    oracle.filter_binomial(D, n, passes, ref)
    eps = 2.0 ** (-24 if prec == "fp32" else -53)
    assert np.abs(np.asarray(J, dtype=np.float64).reshape(3, -1) - ref).max() <= 2 * passes * 3 ** D * eps * scale
    sim.close()
