"""State images and the one-pass reverse: saving and loading a tracked state,
and pic_adjoint_reverse against pic_adjoint_step followed by
pic_adjoint_unpermute from the same state."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    (1, (40,), (8,), 13),
    (2, (24, 16), (8, 8), 5),
    (2, (32, 48), (16, 16), 3),
    (2, (20, 36), (10, 12), 3),
    (3, (8, 8, 12), (4, 8, 6), 2),
    (3, (16, 8, 8), (8, 8, 8), 2),
]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,ppc", CASES)
def test_reverse_from_image_matches_step_and_unpermute(D, n, T, ppc, prec):
    """The particle adjoints are the same arithmetic stored elsewhere: equal
    bit for bit.  The field adjoints sum FP64 LDS atomics in no fixed order and
    round once: 1e-12 (FP64) and 1e-6 (FP32) relative."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, ppc, theta=0.4, seed=40 + D, field_amp=0.05, q=0.01)
    print(f"[gpu] reverse from image D={D} n={n} T={T} {prec}", flush=True)
    sim = PicSim(plasma, tile=T, precision=prec, capacity_factor=3.0, options=L.PIC_OPT_TRACK)
    cap = int(sim.layout.capacity_total)
    sim.step(2, half_b_in_push=True)
    image = sim.save_image()
    before = [sim.particles_host(0, s) for s in range(2)], sim.fields_host(0)
    ids = sim.ids_host()
    gen = torch.Generator(device=sim.device).manual_seed(3)
    rnd = [torch.randn(t.shape, generator=gen, dtype=sim.dtype, device=sim.device) for t in sim.adjoint_buffers()]
    # in place and unpermuted, from the workspace
    lp, lu, lE, lB = (t.clone() for t in rnd)
    pb, ub = torch.zeros_like(lp), torch.zeros_like(lu)
    sim.adjoint_step(lp, lu, lE, lB)
    sim.unpermute(lp, lu, pb, ub, cap)
    # another step changes the workspace; the image does not follow
    sim.step(1, half_b_in_push=True)
    lp2, lu2, lE2, lB2 = (t.clone() for t in rnd)
    pb2, ub2 = torch.zeros_like(lp2), torch.zeros_like(lu2)
    sim.adjoint_reverse(image, lp2, lu2, lE2, lB2, pb2, ub2, cap)
    torch.cuda.synchronize()
    assert torch.equal(pb, pb2) and torch.equal(ub, ub2)
    assert torch.equal(lp2, rnd[0]) and torch.equal(lu2, rnd[1])
    tol = 1e-6 if prec == "fp32" else 1e-12
    for a, b in ((lE, lE2), (lB, lB2)):
        assert float((a - b).norm()) <= tol * float(b.norm())
    # loading the image restores the state
    sim.load_image(image)
    for s in range(2):
        for a, b in zip(before[0][s], sim.particles_host(0, s)):
            assert np.array_equal(a, b)
    for a, b in zip(before[1][:2], sim.fields_host(0)[:2]):
        assert np.array_equal(a, b)
    _, _, _, off, cnt = sim.particle_views()
    used = np.concatenate([np.arange(o, o + c) for o, c in zip(off.reshape(-1).tolist(), cnt.reshape(-1).tolist())])
    assert np.array_equal(sim.ids_host()[used], ids[used])
    assert sim.error() == 0
    with pytest.raises(L.PicError):
        sim.adjoint_reverse(image[4:], lp2, lu2, lE2, lB2, pb2, ub2, cap)     # misaligned image
    sim.close()
