"""Frames that are not tame (gazes far outside the image, extreme parameters) in the passes that
test_gpu_short_math.py does not reach -- reprojected and foveated frames, every compiled slot count -- and what
they cost: they run the same kernels as other frames, only with the general division and root."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2510_03964_amd import fwrs, synth

pytestmark = pytest.mark.gpu
COLOR_TOL = 1e-5     # binary32 weighted mean of at most 16 values in [0, 1] against binary64
GAZES = [(40.0, 20.0), (2.0 ** 25, 7.0), (31.5, 18.5), (1e25, -1e25), (10.25, 30.0), (-3e8, 5.0)]
W, H, DEPTH_TOL = 70, 37, 0.1
BIASES = [fwrs.BIAS_BERNOULLI, fwrs.BIAS_FULL, fwrs.BIAS_MEMORYLESS, fwrs.AES]


def _check(res, orc, out):
    res.sync()
    st, so = res.download(), orc.state()
    for name in ("cnt", "idx"):
        np.testing.assert_array_equal(getattr(st, name), getattr(so, name), err_msg=name)
    for name in ("wsum", "wt", "col", "wslot"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32), err_msg=name)
    assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL


def _pair(k, bias, r2k, flags=0):
    over = dict(fovea_radius_px=9.0, seed=77, stream_id=3, bias_mode=bias, **({} if r2k is None else {"r2k": r2k}))
    res = fwrs.Reservoir(W, H, k, fwrs.default_params(W, **over, flags=flags), stream=torch.cuda.current_stream())
    if not flags and bias in (fwrs.BIAS_BERNOULLI, fwrs.BIAS_MEMORYLESS):
        res.set_resolve_plane_from(2)
    return res, oracle.Oracle(W, H, k, oracle.default_params(W, **over)), torch.full((H, W, 3), -1.0, device="cuda")


@pytest.mark.parametrize("bias", BIASES)
@pytest.mark.parametrize("k,r2k", [(1, None), (2, None), (3, 1e-6), (4, None), (8, 1e-6)])
def test_untame_reprojected_frames_equal_the_oracle(bias, k, r2k):
    spec = synth.StreamSpec(W, H, k, len(GAZES), 9.0, 22.0, 2.0, 3, 4.0)
    src = synth.MovingSource(spec, device="cuda", n_frames=len(GAZES))
    res, orc, out = _pair(k, bias, r2k, fwrs.FLAG_REPROJECT)
    for t, (gx, gy) in enumerate(GAZES):
        c, lev, mv, d, _, _ = src.frame(t)
        res.step_reproject(c, lev, mv, d, gx, gy, DEPTH_TOL, out)
        orc.push_reproject(c.cpu().numpy(), lev.cpu().numpy(), mv.cpu().numpy(), d.cpu().numpy(), gx, gy, DEPTH_TOL)
        _check(res, orc, out)


@pytest.mark.parametrize("mode", [fwrs.FOV_MIP, fwrs.FOV_GAUSS])
@pytest.mark.parametrize("bias", BIASES)
@pytest.mark.parametrize("k,r2k", [(1, None), (2, None), (3, 1e-6), (4, None), (8, 1e-6)])
def test_untame_foveated_frames_equal_the_oracle(mode, bias, k, r2k):
    full = synth.scene(W, H, 3, device="cuda").contiguous()
    res, orc, out = _pair(k, bias, r2k)
    fov = fwrs.Foveator(W, H, 9.0, 22.0, mode, stream=torch.cuda.current_stream())
    for t, (gx, gy) in enumerate(GAZES):
        f = full * (1.0 + 0.03 * t)
        res.step_foveated(fov, f, gx, gy, out)
        orc.push(*oracle.foveate(f.cpu().numpy(), gx, gy, 9.0, 22.0, mode), gx, gy)
        _check(res, orc, out)
    fov.close()


@pytest.mark.parametrize("entry", ["step", "tick", "group"])
@pytest.mark.parametrize("bias", BIASES)
@pytest.mark.parametrize("k,r2k", [(1, None), (2, 1e-6), (8, None)])
def test_untame_frames_at_compiled_slot_counts(entry, bias, k, r2k):
    spec = synth.StreamSpec(W, H, k, len(GAZES), 9.0, 22.0, 2.0, 3, 4.0)
    src = synth.FrameSource(spec, device="cuda")
    res, orc, out = _pair(k, bias, r2k)
    entries = []
    for t, (gx, gy) in enumerate(GAZES):
        c, lev, _, _ = src.frame(t)
        orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
        if entry == "step":
            res.step(c, lev, gx, gy, out)
        else:
            entries.append((res, c, lev, gx, gy, out))
            if entry == "group" and len(entries) < 3:
                continue
            fwrs.tick(entries)
            entries = []
        _check(res, orc, out)


@pytest.mark.parametrize("bias,k,frames", [(fwrs.BIAS_BERNOULLI, 4, 4), (fwrs.BIAS_BERNOULLI, 8, 4), (fwrs.AES, 1, 1)])
def test_untame_sessions_run_the_compiled_kernels(bias, k, frames):
    """A pass over a session of extreme parameters takes at most 1.35 times an ordinary session's: the general
    operations cost a few instructions each (1.0 to 1.1 times), a detour through the run-time slot count or, for
    a group of frames, through memory frame by frame 1.5 to 2.5 times.  Taken in turn, the least of several."""
    w, h = (1280, 720) if frames > 1 else (2560, 1440)
    spec = synth.StreamSpec(w, h, k, 8, 0.05 * w, 0.125 * w, 4.0, 4, 8.0)
    src = synth.FrameSource(spec, device="cuda")
    ring = [src.frame(t) for t in range(8)]
    eng = fwrs.Engine(frames, stream=torch.cuda.current_stream(), use_graph=False)
    best = {}
    ses = {}
    for r2k in (None, 1e-6):
        over = dict(fovea_radius_px=0.05 * w, bias_mode=bias, **({} if r2k is None else {"r2k": r2k}))
        ses[r2k] = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over), stream=torch.cuda.current_stream())
    out = torch.empty((h, w, 3), device="cuda")
    at = 0
    for rep in range(12):
        for r2k, res in ses.items():
            ticks = [[(res, *ring[(at + i * frames + f) % 8], out) for f in range(frames)] for i in range(12)]
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for entries in ticks:
                eng.tick(entries)
            b.record()
            b.synchronize()
            if rep >= 6:
                best[r2k] = min(best.get(r2k, 1e9), a.elapsed_time(b))
        at += 12 * frames
    assert best[1e-6] <= 1.35 * best[None], best
