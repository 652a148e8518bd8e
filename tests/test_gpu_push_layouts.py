"""The push's LDS layouts where the size of a tile decides between them: rows
with the direction codes in LDS, rows with the codes in memory, and planes."""
import numpy as np
import pytest

import oracle
import synth
from oracle import tiles

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,D,n,T", [
    ("fp32", 2, (76, 38), (38, 38)),      # codes in memory: two work-groups, one with them in LDS
    ("fp64", 2, (52, 36), (26, 36)),      # planes: two, one with rows
    ("fp64", 2, (36, 52), (36, 26)),
    ("fp64", 2, (48, 24), (24, 24)),      # codes in memory: three, two
    ("fp64", 2, (18, 36), (18, 18)),
    ("fp32", 3, (8, 12, 6), (4, 6, 6)),
    ("fp64", 1, (2244,), (1122,)),
    ("fp64", 2, (40, 24), (20, 12)),      # rows and codes in LDS
])
@pytest.mark.parametrize("fused", [True, False])
def test_layouts_match_oracle(prec, D, n, T, fused):
    """Two steps of a hot plasma (many leavers) against the oracle from the
    state the GPU holds before each; 1e-12 (FP64) and 1e-5 (FP32) relative L2."""
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, 6, theta=5.0, seed=177 + D, field_amp=0.05, q=0.01)
    print(f"[gpu] push layout D={D} n={n} T={T} {prec} fused={fused}", flush=True)
    sim = PicSim(plasma, tile=T, precision=prec, capacity_factor=4.0)
    st = oracle.State(plasma)
    tol = 1e-5 if prec == "fp32" else 1e-12
    for _ in range(2):
        st.E[:], st.B[:], _ = sim.fields_host(0)
        for s in range(2):
            tid, xl, u = sim.particles_host(0, s)
            st.x[s] = np.ascontiguousarray(tiles.to_global(tid, xl, plasma.n, sim.T, D))
            st.u[s] = np.ascontiguousarray(u.astype(np.float64))
        sim.step(1, fused=fused, half_b_in_push=fused)
        st.step(1)
        assert sim.error() == 0
        for x, y in zip(sim.fields_host(0), (st.E, st.B, st.J)):
            assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    sim.close()
