"""Diagnostics after a state image is loaded describe the loaded state."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,T", [(1, (64,), (8,)), (2, (24, 16), (8, 8)), (3, (8, 8, 12), (4, 8, 6))])
def test_diagnostics_after_load_are_the_images(D, n, T):
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, 6, theta=0.4, seed=31, field_amp=0.05, q=0.01)
    for sp in plasma.species:                  # every third particle on cell corners
        for d in range(D):
            sp.x[d, ::3] = sp.x[d, ::3].round() % n[d]
    sim = PicSim(plasma, tile=T, precision="fp32", capacity_factor=6.0, options=L.PIC_OPT_TRACK)
    before = sim.diagnostics()
    image = sim.save_image()
    assert before["near_face"] > 0
    sim.step(1, half_b_in_push=True)
    assert sim.diagnostics()["near_face"] != before["near_face"]
    sim.step(2, half_b_in_push=True)
    sim.load_image(image)
    after = sim.diagnostics()
    for k in ("particles", "near_face", "error_bits"):
        assert after[k] == before[k], k
    sim.step(2, half_b_in_push=True)
    sim.diagnostics()
    sim.load_image(image)
    sim.step(1, half_b_in_push=True)           # one step, but from another state than the last diagnostics
    assert sim.diagnostics()["continuity_max"] == -1
    sim.step(1, half_b_in_push=True)
    assert 0 <= sim.diagnostics()["continuity_max"] < 1e-5
    sim.close()
