"""Reverse windows of a simulation with a stream of its own, called from
another one: checkpoints, adjoints and results are ordered with the steps."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("particles", [False, True])
def test_windows_on_another_stream(particles):
    """FP32 steps repeat bit for bit; the field adjoints sum FP64 LDS atomics
    in no fixed order and round once a step (1e-6 relative)."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd import adjoint
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(2, (96, 64), 40, theta=0.4, seed=19, field_amp=0.05, q=1e-3)
    got = []
    for stream in (None, torch.cuda.Stream()):
        sim = PicSim(plasma, tile=(8, 8), precision="fp32", capacity_factor=3.0, options=L.PIC_OPT_TRACK, stream=stream)
        torch.cuda.synchronize()
        cap = int(sim.layout.capacity_total)
        ck = adjoint.forward(sim, 6, window=3)
        E, B, _ = (t.clone() for t in sim.field_views())       # behind forward on the caller's stream
        lp = torch.ones((2, cap), device=sim.device) if particles else None
        out = adjoint.backward(sim, ck, 6, 2 * E, B, lpos=lp, window=3)
        del ck, lp
        junk = [torch.full((3, cap), 7.0, device=sim.device) for _ in range(8)]   # over freed checkpoints and buffers
        got.append([E, B] + [t.clone() for t in out])
        del junk, out
        assert sim.error() == 0
        sim.close()
    for a, b in zip(*got):
        assert float((a - b).norm()) <= 1e-6 * float(b.norm())
