"""GPU current filter with several passes per launch against the oracle: odd
and even pass counts, boxes shorter than the halo of a launch, tiles that are
not a power of two, and tiles whose block does not fit the LDS."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,tile,passes", [
    (1, (8,), (8,), 11),                # halo as long as the box
    (1, (40,), (10,), 17),              # three launches become four
    (2, (48, 24), (12, 8), 3),
    (2, (40, 32), (20, 16), 5),
    (2, (4, 4), (4, 4), 7),
    (3, (16, 8, 24), (8, 8, 8), 2),
    (3, (16, 8, 24), (8, 8, 8), 5),
    (3, (16, 16, 16), (16, 16, 16), 3),  # FP64 block of 18^3 cells: straight from memory
])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_filter_passes_match_oracle(D, n, tile, passes, prec):
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
    # a pass rounds a sum of at most 3^D terms of weight 1 in all; the weights
    # are powers of two
    eps = 2.0 ** (-24 if prec == "fp32" else -53)
    assert np.abs(np.asarray(J, dtype=np.float64).reshape(3, -1) - ref).max() <= 2 * passes * 3 ** D * eps * scale
    sim.close()
