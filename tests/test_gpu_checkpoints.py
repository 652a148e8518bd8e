"""Checkpoints in either form: state images (what adjoint.forward returns)
and the workspace copies of PicSim.snapshot."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def tracked():
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(2, (24, 16), 5, theta=0.4, seed=12, field_amp=0.05, q=0.01)
    return PicSim(plasma, tile=(8, 8), precision="fp32", capacity_factor=4.0, options=L.PIC_OPT_TRACK)


def state(sim):
    return [*sim.fields_host(0)[:2], *(a for s in range(2) for a in sim.particles_host(0, s))]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b, strict=True))


def test_restore_takes_either_form():
    from paper_1906_06306_amd import adjoint
    sim = tracked()
    start, snap = state(sim), sim.snapshot()
    ck = adjoint.forward(sim, 4, window=2)
    assert not same(state(sim), start)
    sim.restore(snap)
    assert same(state(sim), start)
    sim.step(2, half_b_in_push=True)
    mid = state(sim)
    sim.restore(ck[0])
    assert same(state(sim), start)
    sim.restore(ck[2])
    assert same(state(sim), mid)
    assert sim.error() == 0
    sim.close()


def test_backward_takes_snapshots():
    """FP32 steps repeat bit for bit, so both forms give the same sweep; the
    field adjoints sum FP64 LDS atomics in no fixed order (1e-6 relative, as
    for one reversed step)."""
    from paper_1906_06306_amd import adjoint
    sim = tracked()
    ck = adjoint.forward(sim, 5, window=2)
    E, B, _ = (t.clone() for t in sim.field_views())
    want = adjoint.backward(sim, ck, 5, E, B, window=2)
    snaps = {}
    for k in ck:
        sim.restore(ck[k])
        snaps[k] = sim.snapshot()
    got = adjoint.backward(sim, snaps, 5, E, B, window=2)
    assert sim.error() == 0
    for a, b in zip(got, want):
        assert float((a - b).norm()) <= 1e-6 * float(b.norm())
    sim.close()


@pytest.mark.parametrize("bad", [0, 2])
def test_backward_from_snapshots_reports_a_rejected_origin(bad):
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd import adjoint
    sim = tracked()
    snaps = {0: sim.snapshot()}
    sim.step(2, half_b_in_push=True)
    snaps[2] = sim.snapshot()
    sim.step(2, half_b_in_push=True)
    E, B, _ = (t.clone() for t in sim.field_views())
    sim.restore(snaps[bad])
    sim.ids_view()[int(sim.particle_views()[3][3, 0])] = -1
    snaps[bad] = sim.snapshot()
    assert sim.error() == 0
    adjoint.backward(sim, snaps, 4, E, B, window=2)
    assert sim.error() == L.PIC_E_ADJ_MAP
    sim.close()
