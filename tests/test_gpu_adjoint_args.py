"""What the one-pass reverse and the state images refuse."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture()
def sim():
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    s = PicSim(synth.small_random(2, (24, 16), 3, seed=4, field_amp=0.05), tile=(8, 8), precision="fp32",
               capacity_factor=4.0, options=L.PIC_OPT_TRACK)
    yield s
    s.close()


def test_reverse_refuses_overlapping_particle_adjoints(sim):
    from paper_1906_06306_amd import _lib as L
    image = sim.save_image()
    sim.step(1, half_b_in_push=True)
    cap = int(sim.layout.capacity_total)
    _, _, lE, lB = sim.adjoint_buffers()
    # the four particle buffers as parts of one block, side by side
    block = torch.zeros(10 * cap, dtype=sim.dtype, device=sim.device)
    part = lambda plane, planes: block[plane * cap:(plane + planes) * cap].view(planes, cap)
    lp, lu, pb, ub = part(0, 2), part(2, 3), part(5, 2), part(7, 3)
    sim.adjoint_reverse(image, lp, lu, lE, lB, pb, ub, cap)
    for bad in ((lp, lu, lp, ub), (lp, lu, pb, lu), (lp, lu, part(1, 2), ub), (lp, lu, part(3, 2), ub),
                (lp, lu, pb, part(1, 3)), (lp, lu, pb, part(6, 3))):
        with pytest.raises(L.PicError) as e:
            sim.adjoint_reverse(image, bad[0], bad[1], lE, lB, bad[2], bad[3], cap)
        assert e.value.code == L.PIC_E_ARG
    assert sim.error() == 0


def test_images_of_another_size_are_refused(sim):
    from paper_1906_06306_amd import _lib as L
    image = sim.save_image()
    la, ua, lE, lB = sim.adjoint_buffers()
    pb, ub, _, _ = sim.adjoint_buffers()
    for bad in (image[:-256], image.view(torch.int32), torch.stack([image, image])[:, ::2], image.cpu()):
        for call in (lambda: sim.save_image(bad), lambda: sim.load_image(bad),
                     lambda: sim.adjoint_reverse(bad, la, ua, lE, lB, pb, ub, int(sim.layout.capacity_total))):
            with pytest.raises(L.PicError) as e:
                call()
            assert e.value.code == L.PIC_E_ARG
    sim.load_image(image)
    assert sim.error() == 0
