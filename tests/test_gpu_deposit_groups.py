"""The unfused deposit's groups of particles per lane (four; two in 3D FP64)
against the oracle, for segments that end anywhere in a group or a wave."""
import numpy as np
import pytest

import oracle
import synth
from oracle import tiles

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,ppc", [
    (1, (48,), (8,), 60),
    (2, (24, 16), (8, 4), 12),
    (3, (8, 8, 8), (4, 4, 4), 7),
    (3, (8, 12, 8), (8, 6, 8), 3),
])
def test_deposit_of_uneven_segments(D, n, T, ppc, prec):
    """Segments of 0, 1, 2, ... particles up to the full count; tolerances are
    the 1e-12 (FP64) and 1e-5 (FP32) relative L2 of the method."""
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, ppc, theta=0.5, seed=90 + D, field_amp=0.05, q=0.01)
    for k, sp in enumerate(plasma.species):
        tile = np.zeros(sp.x.shape[1], dtype=np.int64)
        for d in range(D):
            tile = tile * (n[d] // T[d]) + (sp.x[d] // T[d]).astype(np.int64)
        rank = np.empty_like(tile)
        for t in range(tile.max() + 1):
            at = np.flatnonzero(tile == t)
            rank[at] = np.arange(at.size)
        most = np.array([0, 1, 2, 3, 5, 63, 64, 65, 127, 129, 130, 255])
        keep = rank < most[(tile + 3 * k) % most.size]
        sp.x, sp.u = np.ascontiguousarray(sp.x[:, keep]), np.ascontiguousarray(sp.u[:, keep])
    print(f"[gpu] uneven deposit D={D} T={T} {prec}", flush=True)
    sim = PicSim(plasma, tile=T, precision=prec, capacity_factor=20.0)
    st = oracle.State(plasma)
    st.E[:], st.B[:], _ = sim.fields_host(0)
    for s in range(2):
        tid, xl, u = sim.particles_host(0, s)
        st.x[s] = np.ascontiguousarray(tiles.to_global(tid, xl, plasma.n, sim.T, D))
        st.u[s] = np.ascontiguousarray(u.astype(np.float64))
    sim.step(1, fused=False)
    st.step(1)
    assert sim.error() == 0
    tol = 1e-5 if prec == "fp32" else 1e-12
    for x, y in zip(sim.fields_host(0), (st.E, st.B, st.J)):
        assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    sim.close()
