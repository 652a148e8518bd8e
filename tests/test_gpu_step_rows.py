"""Fused steps with FDTD4 or the current filter, whose rows share launches,
against the stages called one by one: bit for bit, at tiles that leave waves
idle, boxes of one tile, odd pass counts and several boxes."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half_b_in_push", [False, True])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("D,n,T,kw", [
    (1, (12,), (4,), dict(fdtd_order=4)),
    (1, (40,), (10,), dict(filter_passes=3)),
    (2, (8, 8), (8, 8), dict(fdtd_order=4, filter_passes=1)),
    (2, (60, 36), (20, 12), dict(fdtd_order=4, filter_passes=8)),
    (2, (32, 16), (8, 8), dict(filter_passes=5, pusher="hc")),
    (3, (16, 8, 12), (8, 4, 6), dict(fdtd_order=4, filter_passes=2)),
])
def test_step_matches_stages(D, n, T, kw, prec, half_b_in_push):
    from paper_1906_06306_amd import _lib as L
    from paper_1906_06306_amd.sim import PicSim
    boxes = [synth.small_random(D, n, 4, theta=0.4, seed=60 + k, field_amp=0.05, q=0.01) for k in range(2)]
    a = PicSim(boxes, tile=T, precision=prec, capacity_factor=4.0, **kw)
    b = PicSim(boxes, tile=T, precision=prec, capacity_factor=4.0, **kw)
    second = kw.get("fdtd_order", 2) == 2 and half_b_in_push   # FDTD4 keeps half B out of the push
    a.step(3, half_b_in_push=half_b_in_push)
    for _ in range(3):
        if not second:
            b.fdtd(L.PIC_HALF_B)
        b.push(half_b=second)
        b.fdtd(L.PIC_TWO_HALF_B if second else L.PIC_HALF_B)
        b.deposit()
        if kw.get("filter_passes"):
            b.filter_current(kw["filter_passes"])
        b.fdtd(L.PIC_CURL_E_ADD_J)
        b.sort_migrate()
    assert a.error() == 0 and b.error() == 0
    # FP64 currents are summed in no fixed order: 3 steps of at most 2^10
    # additions of 2^-53; FP32 sums are exact
    tol = 0.0 if prec == "fp32" else 3 * 2.0 ** -43
    for k in range(2):
        for x, y in zip(a.fields_host(k), b.fields_host(k)):
            x, y = np.asarray(x), np.asarray(y)
            assert np.abs(x - y).max() <= tol * np.abs(y).max()
        for s in range(2):
            for x, y in zip(a.particles_host(k, s), b.particles_host(k, s)):
                x, y = np.asarray(x), np.asarray(y)
                assert x.shape == y.shape and np.abs(x - y).max() <= tol * max(1.0, np.abs(y).max())
    a.close()
    b.close()
