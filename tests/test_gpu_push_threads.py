"""The push's work-group size: exactly the block on request, otherwise what
the library reports, with the same results."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,ppc", [(1, (64,), (16,), 100), (2, (32, 32), (16, 16), 12), (3, (16, 16, 8), (8, 8, 8), 4)])
def test_exact_block(D, n, T, ppc, prec, persistent):
    """Few segments of over 1,024 particles: the library takes more threads
    than asked, and the exact block when told to.  FP32 states agree bit for
    bit; FP64 currents sum in the order the waves reach them (1e-12)."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, ppc, theta=0.5, seed=21, field_amp=0.05, q=0.01)
    walker = L.PIC_OPT_PERSISTENT if persistent else 0
    print(f"[gpu] push threads D={D} {prec} persistent={persistent}", flush=True)
    got = []
    for block, opt in ((64, L.PIC_OPT_EXACT_BLOCK), (256, L.PIC_OPT_EXACT_BLOCK), (64, 0)):
        sim = PicSim(plasma, tile=T, precision=prec, block=block, capacity_factor=3.0, options=opt | walker)
        assert sim.push_threads() == 0 and sim.push_threads(fused=False) == 0
        sim.step(3, half_b_in_push=True)
        assert sim.push_threads(fused=False) == 0
        if opt:
            assert sim.push_threads() == block
        else:
            assert block < sim.push_threads() <= 1024
        sim.step(1, fused=False)
        assert (sim.push_threads(fused=False) == block) or not opt
        assert sim.error() == 0
        got.append([*sim.fields_host(0), *(a for s in range(2) for a in sim.particles_host(0, s))])
        sim.close()
    tol = 0.0 if prec == "fp32" else 1e-12
    for other in got[:2]:
        for a, b in zip(other, got[2], strict=True):
            assert np.abs(a - b).max() <= tol * max(1.0, np.abs(b).max())


@pytest.mark.parametrize("T,raised", [((6, 6, 6), False), ((8, 8, 8), True)])
def test_many_segments_keep_the_block_unless_waves_grow_by_half(T, raised):
    """FP64, more segments than two rounds of resident groups: 6^3 tiles hold
    12 waves of 256 threads on a CU and 16 of 512, 8^3 tiles 4 and 16."""
    from paper_1906_06306_amd.sim import PicSim
    n = tuple(12 * t for t in T)
    sim = PicSim(synth.small_random(3, n, 5, theta=0.3, seed=2), tile=T, precision="fp64", block=256,
                 capacity_factor=1.6)
    sim.step(1, half_b_in_push=True)
    assert (sim.push_threads() > 256) == raised
    assert sim.error() == 0
    sim.close()
