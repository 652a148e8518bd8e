"""The whole step's two launches (push, then fold + E + B + arrivals) against
the stages called one by one, at the tile shapes where the fold's neighbour
walk and the arrivals can go wrong: edges of 2 and 4 (a cell covered from both
sides), boxes of one or two tiles (a tile is its own neighbour), ragged tiles,
walls, and several boxes in one batch."""
import numpy as np
import pytest

import oracle
import synth
from oracle import tiles

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [
    (1, (6,), (2,), False),
    (1, (8,), (8,), True),
    (2, (8, 8), (8, 8), False),
    (2, (12, 8), (2, 4), False),
    (2, (60, 36), (20, 12), True),
    (3, (8, 4, 6), (4, 4, 2), False),
    (3, (16, 8, 8), (8, 8, 8), True),
    (3, (8, 16, 24), (8, 8, 8), False),
]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,walls", SHAPES)
def test_whole_step_matches_stages(D, n, T, walls, prec):
    """Four steps.  FP32 current sums are exact integers and every other
    operation has a fixed order, so FP32 states agree bit for bit; FP64
    current blocks sum in the order the waves reach them, which leaves a few
    units of 1e-16 per step (bound 1e-12)."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    plasmas = [synth.small_random(D, n, 5, theta=1.0, seed=500 + k, field_amp=0.05, q=0.01) for k in range(2)]
    print(f"[gpu] whole step D={D} n={n} T={T} walls={walls} {prec}", flush=True)
    a, b = (PicSim(plasmas, tile=T, precision=prec, walls=walls, capacity_factor=4.0) for _ in range(2))
    for _ in range(4):
        a.step(1, fused=True, half_b_in_push=True)
        b.push(fused=True, half_b=True)
        b.fdtd(L.PIC_TWO_HALF_B)
        b.deposit()
        b.fdtd(L.PIC_CURL_E_ADD_J)
        b.sort_migrate()
    assert a.error() == 0 and b.error() == 0
    tol = 0.0 if prec == "fp32" else 1e-12
    for box in range(2):
        for x, y in zip(a.fields_host(box), b.fields_host(box)):
            assert np.abs(x - y).max() <= tol * max(1.0, np.abs(y).max())
        for s in range(2):
            pa, pb = a.particles_host(box, s), b.particles_host(box, s)
            assert np.array_equal(pa[0], pb[0])
            assert np.abs(pa[1] - pb[1]).max() <= tol and np.abs(pa[2] - pb[2]).max() <= tol * np.abs(pb[2]).max()
    a.close()
    b.close()


LAYOUTS = [
    # (D, n, T, ppc): rows of six components with a constant edge, padded
    # rows, rows with runtime edges, and the largest tile of two FP64 edges,
    # whose rows do not fit the LDS (one plane per component)
    (1, (64,), (32,), 9),
    (2, (32, 16), (16, 16), 5),
    (2, (32, 64), (32, 32), 3),
    (2, (40, 36), (20, 12), 4),
    (2, (96, 84), (48, 42), 2),
    (3, (16, 8, 16), (8, 8, 8), 3),
    (3, (12, 10, 8), (6, 10, 4), 3),
]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,ppc", LAYOUTS)
def test_field_layouts_match_oracle(D, n, T, ppc, prec):
    """One whole step from the state the GPU holds, against the FP64 oracle,
    for every way the push lays out E, B and the current in LDS.  Tolerances:
    the 1e-12 (FP64) and 1e-5 (FP32) relative L2 of the method."""
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, ppc, theta=0.5, seed=77 + D, field_amp=0.05, q=0.01)
    print(f"[gpu] layout D={D} n={n} T={T} {prec}", flush=True)
    sim = PicSim(plasma, tile=T, precision=prec, capacity_factor=4.0)
    st = oracle.State(plasma)
    st.E[:], st.B[:], _ = sim.fields_host(0)
    for s in range(2):
        tid, xl, u = sim.particles_host(0, s)
        st.x[s] = np.ascontiguousarray(tiles.to_global(tid, xl, plasma.n, sim.T, D))
        st.u[s] = np.ascontiguousarray(u.astype(np.float64))
    sim.step(1, half_b_in_push=True)
    st.step(1)
    assert sim.error() == 0
    tol = 1e-5 if prec == "fp32" else 1e-12
    for x, y in zip(sim.fields_host(0), (st.E, st.B, st.J)):
        assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    sim.close()


@pytest.mark.parametrize("kw", [{}, dict(fdtd_order=4), dict(filter_passes=2)])
def test_whole_step_refuses_cell_sort_with_tracking(kw):
    """The cell sort does not record origins: a tracked step with it is an
    error however the step is launched."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    sim = PicSim(synth.small_random(2, (32, 16), 3, seed=5), tile=(8, 8), precision="fp32", options=L.PIC_OPT_TRACK,
                 **kw)
    flags = L.PIC_FUSED | L.PIC_PUSH_HALF_B | L.PIC_SORT_CELLS
    assert L.lib().pic_step(sim.ctx, flags) == L.PIC_E_ARG
    sim.close()
