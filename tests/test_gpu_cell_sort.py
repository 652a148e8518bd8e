"""The cell sort where its paths change: segments permuted through LDS, larger
ones scattered to the staging planes, tiles of so many cells that half the
waves sort them, an empty species, counts that are no multiple of a wave."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # (D, n, T, ppc)
    (1, (48,), (16,), 5),
    (1, (6000,), (3000,), 3),          # 3,000 cells: 4 waves, through LDS
    (2, (24, 40), (8, 20), 7),
    (2, (8, 8), (8, 8), 129),          # 8,256 particles: staging planes
    (2, (96, 48), (48, 48), 4),        # 2,304 cells and 9,216 particles: both
    (3, (8, 16, 6), (8, 8, 6), 11),
]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,ppc", CASES)
def test_cell_sort_is_stable_and_exact(D, n, T, ppc, prec):
    """Between steps, the sort permutes every segment by the stable order of
    its cell indices (x fastest): positions and momenta equal the permuted
    ones bit for bit."""
    from paper_1906_06306_amd.sim import PicSim
    plasma = synth.small_random(D, n, ppc, theta=0.4, seed=900 + D)
    plasma.species[1].x = plasma.species[1].x[:, :0]
    plasma.species[1].u = plasma.species[1].u[:, :0]
    print(f"[gpu] cell sort D={D} n={n} T={T} {prec}", flush=True)
    sim = PicSim(plasma, tile=T, precision=prec, capacity_factor=2.0)
    tid, x, u = sim.particles_host(0, 0)
    near = sim.diagnostics()["near_face"]
    sim.sort_migrate(sort_cells=True)
    tid2, x2, u2 = sim.particles_host(0, 0)
    key = np.zeros(tid.size, dtype=np.int64)
    stride = 1
    for d in range(D):
        key += (np.floor(x[d]).astype(np.int64) + T[d] // 2) * stride
        stride *= T[d]
    order = np.lexsort((np.arange(tid.size), key, tid))
    assert np.array_equal(tid2, tid[order])
    assert np.array_equal(x2, x[:, order]) and np.array_equal(u2, u[:, order])
    d = sim.diagnostics()
    assert d["status"] == 0 and d["near_face"] == near
    sim.close()
