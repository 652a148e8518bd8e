"""adjoint.backward with particle adjoints, from whatever state the workspace
holds on entry: a second loss over the same checkpoints, or a simulation that
has stepped on."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def used_slots(sim):
    _, _, _, off, cnt = sim.particle_views()
    return np.concatenate([np.arange(o, o + c) for o, c in zip(off.reshape(-1).tolist(), cnt.reshape(-1).tolist())])


@pytest.mark.parametrize("nsteps,window", [(1, 8), (3, 8), (4, 2), (5, 2)])
def test_backward_does_not_depend_on_the_state_held(nsteps, window):
    """FP64 against the oracle's adjoint (relative L2 1e-10, as for one step):
    from the final state, from the initial state that the first call leaves,
    and from a state two steps on."""
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd import adjoint
    from paper_1906_06306_amd.sim import PicSim
    n, T = (24, 16, 1), (8, 8)
    plasma = synth.small_random(2, n, 4, seed=77, field_amp=0.05, q=0.02)
    sim = PicSim(plasma, tile=T, precision="fp64", capacity_factor=3.0, options=L.PIC_OPT_TRACK)
    print(f"[gpu] backward from any state, {nsteps} steps, windows of {window}", flush=True)
    rng = np.random.default_rng(3)
    npart = [sp.x.shape[1] for sp in plasma.species]
    lx, lu = ([rng.standard_normal((d, k)) for k in npart] for d in (2, 3))
    lE, lB = rng.standard_normal((2, 3, n[0] * n[1]))
    # adjoints of the final particles, placed at their slots: the origin ids
    # of every step lead from a final slot to the input index
    probe = PicSim(plasma, tile=T, precision="fp64", capacity_factor=3.0, options=L.PIC_OPT_TRACK)
    inp = probe.ids_host().copy()
    for _ in range(nsteps):
        probe.step(1, half_b_in_push=True)
        slots, before = used_slots(probe), inp
        inp = np.full_like(before, -1)
        inp[slots] = before[probe.ids_host()[slots]]
    probe.close()
    inp = inp[slots]
    assert np.array_equal(np.sort(inp), np.arange(sum(npart)))
    la, ua, _, _ = sim.adjoint_buffers()
    for t, v in ((la, lx), (ua, lu)):
        t[:, torch.as_tensor(slots, device=sim.device)] = torch.as_tensor(np.concatenate(v, axis=1)[:, inp],
                                                                          device=sim.device)
    dev = [torch.as_tensor(v, device=sim.device) for v in (lE, lB)]
    # the oracle, step by step backwards from its own states
    states = [oracle.State(plasma)]
    for _ in range(nsteps - 1):
        states.append(states[-1].copy())
        states[-1].step(1)
    for st in reversed(states):
        st.step_adjoint(lx, lu, lE, lB)
    ck = adjoint.forward(sim, nsteps, window)
    sl = sim.input_slices()
    for entry in ("final", "initial", "later"):
        if entry == "later":
            sim.step(nsteps + 2, half_b_in_push=True)
        out = adjoint.backward(sim, ck, nsteps, *dev, lpos=la, lu=ua, window=window)
        g_x, g_u, g_E, g_B = (t.cpu().numpy() for t in out)
        assert sim.error() == 0
        assert rel(g_E, lE) < 1e-10 and rel(g_B, lB) < 1e-10, entry
        for s in range(2):
            assert rel(g_x[:, sl[(0, s)]], lx[s]) < 1e-10, (entry, s)
            assert rel(g_u[:, sl[(0, s)]], lu[s]) < 1e-10, (entry, s)
    sim.close()
