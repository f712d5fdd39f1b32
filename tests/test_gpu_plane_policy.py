"""Frames from the resolve plane on either side of the size (256 MiB of slot records in a launch) at which the
plane's cache policy changes, through every pass that has the choice, with short and long lists of changed pixels
and the slot counts that load colours with one lane per pixel."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2510_03964_amd import fwrs, synth

pytestmark = pytest.mark.gpu
COLOR_TOL = 1e-5     # binary32 weighted mean of at most 16 values in [0, 1] against binary64


def _session(w, h, k, sid):
    over = dict(fovea_radius_px=0.05 * w, seed=synth.PHILOX_SEED, stream_id=sid)
    res = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over), stream=torch.cuda.current_stream())
    res.set_resolve_plane_from(2)
    return res, oracle.Oracle(w, h, k, oracle.default_params(w, **over)), torch.full((h, w, 3), -1.0, device="cuda")


def _check(res, orc, out):
    st, so = res.download(), orc.state()
    np.testing.assert_array_equal(st.idx, so.idx)
    for name in ("wsum", "wt", "col"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32))
    assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL


@pytest.mark.parametrize("entry,w,h,k,sessions", [
    ("step", 1024, 1024, 16, 1), ("step", 1024, 1025, 16, 1), ("step", 2048, 1025, 8, 1), ("step", 63, 37, 8, 1),
    ("step", 67, 35, 16, 1), ("tick", 1024, 1024, 8, 2), ("tick", 1024, 1025, 8, 2), ("tick", 67, 35, 5, 2),
    ("mip", 1024, 1024, 16, 1), ("mip", 1024, 1025, 16, 1), ("gauss", 65, 37, 8, 1), ("mip", 63, 33, 2, 1)])
def test_plane_frames(entry, w, h, k, sessions):
    n = 5
    spec = synth.StreamSpec(w, h, k, n, 0.05 * w, 0.125 * w, 2.0, 2, 6.0)
    ses = [_session(w, h, k, 3 + i) for i in range(sessions)]
    if entry in ("mip", "gauss"):
        mode = fwrs.FOV_MIP if entry == "mip" else fwrs.FOV_GAUSS
        fov = fwrs.Foveator(w, h, 0.05 * w, 0.125 * w, mode, stream=torch.cuda.current_stream())
        full = synth.scene(w, h, 3, device="cuda").contiguous()
        gaze = synth.gaze_trace(spec, n)
        res, orc, out = ses[0]
        for t in range(n):
            gx, gy = float(gaze[t, 0]), float(gaze[t, 1])
            f = full * (1.0 + 0.05 * t)
            res.step_foveated(fov, f, gx, gy, out)
            orc.push(*oracle.foveate(f.cpu().numpy(), gx, gy, 0.05 * w, 0.125 * w, mode), gx, gy)
        fov.close()
    else:
        src = synth.FrameSource(spec, device="cuda")
        for t in range(n):
            c, lev, gx, gy = src.frame(t)
            if entry == "step":
                ses[0][0].step(c, lev, gx, gy, ses[0][2])
            else:
                fwrs.tick([(res, c, lev, gx, gy, out) for res, _, out in ses])
            for _, orc, _ in ses:
                orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
    for res, orc, out in ses:
        res.sync()
        _check(res, orc, out)
