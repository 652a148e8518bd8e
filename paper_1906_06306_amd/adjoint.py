"""Reverse mode over windows of fused steps, with checkpointed recomputation.

The forward run keeps an image of the state (fields, the particles in use,
segment counts, origin ids) every ``window`` steps.  The reverse sweep visits
the windows last to first: it loads the window's checkpoint, re-runs the
window keeping an image of every state, and then, step by step backwards,
applies the step's transposed Jacobian from that image and moves the particle
adjoints across the migration of the step before it
(``pic_adjoint_reverse``, with the origin ids of the image).  After the first
step the particle adjoints are in the input order of ``pic_init_tiles``.  All
arithmetic runs in the library's kernels; this module only orders the calls.

``PicWindow`` wraps one box as a ``torch.autograd.Function`` of its initial
state (positions, four-velocities, E, B), so that gradients of any loss of
the final fields with respect to parameters of the initial state follow
from autograd.
"""
from __future__ import annotations

import contextlib

import torch

from . import _lib as L
from .sim import Box, PicSim

STEP_FLAGS = L.PIC_FUSED | L.PIC_PUSH_HALF_B


@contextlib.contextmanager
def _sim_stream(sim: PicSim):
    """torch's allocations, copies and fills on the simulation's stream, behind
    the caller's work and ahead of the caller's next."""
    cur = torch.cuda.current_stream(sim.device)
    if cur == sim.stream:
        yield
        return
    sim.stream.wait_stream(cur)
    with torch.cuda.stream(sim.stream):
        yield
    cur.wait_stream(sim.stream)


def forward(sim: PicSim, nsteps: int, window: int = 8) -> dict:
    """Run nsteps tracked fused steps; return {step: state image} at the
    window starts."""
    if not sim.cfg.options & L.PIC_OPT_TRACK:
        raise ValueError("the simulation needs options=PIC_OPT_TRACK")
    fn = L.lib().pic_step
    with _sim_stream(sim):
        ckpts = {0: sim.save_image()}
        for k in range(nsteps):
            L.check(fn(sim.ctx, STEP_FLAGS))
            if (k + 1) % window == 0 and k + 1 < nsteps:
                ckpts[k + 1] = sim.save_image()
    return ckpts


def _load(sim: PicSim, ckpt) -> torch.Tensor:
    """Load a checkpoint, keeping the error bits latched so far; its image."""
    if isinstance(ckpt, torch.Tensor):
        sim.load_image(ckpt)
        return ckpt
    word = sim.error_view()
    bits = word.clone()
    sim.restore(ckpt)
    word |= bits
    return sim.save_image()


def backward(sim: PicSim, ckpts: dict, nsteps: int, lE, lB, lpos=None, lu=None, window: int = 8):
    """Adjoints of the initial state from those of the state after nsteps.

    ckpts: {step: checkpoint} as from ``forward``, each a state image or a
    ``PicSim.snapshot()``.
    lE, lB: (3, cells_total) adjoints of E^N, B^{N-1/2}; lpos, lu: adjoints
    of the final particles in the final state's slots (zero if None).  The
    simulation may hold any state on entry (for nsteps = 0 the final one).
    Returns (lpos_in (D, n_input), lu_in (3, n_input), lE0, lB0) in the
    working precision, the particle adjoints in the concatenated input order.
    Leaves the initial state in the workspace, and every error bit that the
    sweep latched: with one of them (``sim.error()``) the adjoints are not
    valid."""
    with _sim_stream(sim):
        out = _sweep(sim, ckpts, nsteps, lE, lB, lpos, lu, window)
    for t in out:
        t.record_stream(torch.cuda.current_stream(sim.device))
    return out


def _sweep(sim: PicSim, ckpts: dict, nsteps: int, lE, lB, lpos, lu, window: int):
    fn = L.lib().pic_step
    la, ua, _, _ = sim.adjoint_buffers()
    lb, ub, _, _ = sim.adjoint_buffers()
    lE = lE.to(sim.dtype).contiguous().clone()
    lB = lB.to(sim.dtype).contiguous().clone()
    cap = int(sim.layout.capacity_total)
    n_in = sim.n_input
    lpos_in = torch.zeros((sim.D, n_in), dtype=sim.dtype, device=sim.device)
    lu_in = torch.zeros((3, n_in), dtype=sim.dtype, device=sim.device)
    particles = lpos is not None or lu is not None
    if lpos is not None:
        la.copy_(lpos)
    if lu is not None:
        ua.copy_(lu)
    if particles and nsteps == 0:
        sim.unpermute(la, ua, lpos_in, lu_in, n_in)
    images = []                            # of the states inside a window
    for w0 in sorted((k for k in ckpts if k < nsteps), reverse=True):
        w1 = min(w0 + window, nsteps)
        start = _load(sim, ckpts[w0])
        for j in range(w0 + 1, w1):
            L.check(fn(sim.ctx, STEP_FLAGS))
            if len(images) < j - w0:
                images.append(sim.new_image())
            sim.save_image(images[j - w0 - 1])
        if particles:
            # to the slots of the state before the last step, by the origin
            # ids of the state after it: that step is run again, since the
            # workspace may hold any state on entry
            L.check(fn(sim.ctx, STEP_FLAGS))
            sim.unpermute(la, ua, lb, ub, cap)
            particles = False
        for k in range(w1 - 1, w0 - 1, -1):
            state = start if k == w0 else images[k - w0 - 1]
            out = (lpos_in, lu_in, n_in) if k == 0 else (la, ua, cap)
            sim.adjoint_reverse(state, lb, ub, lE, lB, *out)
            la, lb = lb, la
            ua, ub = ub, ua
    if nsteps and 0 in ckpts:
        sim.load_image(start)
    return lpos_in, lu_in, lE, lB


class PicWindow(torch.autograd.Function):
    """E^N, B^{N-1/2} of one box after nsteps fused steps, as a function of
    the initial state.  Inputs after the settings: E0 (3, N), B0 (3, N) and
    per species pos (D, np), u (3, np), all FP64 tensors on the device."""

    @staticmethod
    def forward(ctx, settings: dict, E0, B0, *parts):
        ns = len(parts) // 2
        box = Box(D=settings["D"], n=tuple(settings["n"]), c=settings["c"], charge=list(settings["charge"]),
                  qm=list(settings["qm"]), mass=list(settings["mass"]), pos=list(parts[0::2]),
                  u=list(parts[1::2]), E=E0, B=B0)
        sim = PicSim(box, tile=settings["tile"], precision=settings.get("precision", "fp32"),
                     capacity_factor=settings.get("capacity_factor", 2.0), options=L.PIC_OPT_TRACK,
                     device=str(E0.device))
        nsteps, window = int(settings["nsteps"]), int(settings.get("window", 8))
        ckpts = forward(sim, nsteps, window)
        E, B, _ = sim.field_views()
        err = sim.error()
        if err:
            raise L.PicError(err, L.lib().pic_last_error().decode())
        ctx.sim, ctx.ckpts, ctx.nsteps, ctx.window, ctx.ns = sim, ckpts, nsteps, window, ns
        return E.to(torch.float64).clone(), B.to(torch.float64).clone()

    @staticmethod
    def backward(ctx, gE, gB):
        sim = ctx.sim
        z = torch.zeros((3, int(sim.layout.cells_total)), dtype=torch.float64, device=sim.device)
        gE = z if gE is None else gE
        gB = z if gB is None else gB
        lpos, lu, lE, lB = backward(sim, ctx.ckpts, ctx.nsteps, gE, gB, window=ctx.window)
        err = sim.error()
        if err:
            raise L.PicError(err, L.lib().pic_last_error().decode())
        grads = [None, lE.double(), lB.double()]
        for (b, s), sl in sim.input_slices().items():
            grads += [lpos[:, sl].double(), lu[:, sl].double()]
        sim.close()
        ctx.sim = ctx.ckpts = None
        return tuple(grads)
