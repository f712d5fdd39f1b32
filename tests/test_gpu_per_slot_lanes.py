"""The per-slot modes (Eq. 7, A-ES) through every pass and both forms -- one lane per pixel and one lane per
slot -- with colours that change everywhere, change in part of a wave, or hold still, so that the new colour's
Lab is needed by all, some or none of a wave's slots; and a store above 256 MiB."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2510_03964_amd import fwrs, synth

pytestmark = pytest.mark.gpu
COLOR_TOL = 1e-5     # binary32 weighted mean of at most 16 values in [0, 1] against binary64
DEPTH_TOL = 0.1


def _colours(base, t, kind):
    if kind == "still":
        return base
    g = torch.Generator().manual_seed(100 + t)
    noise = torch.rand(base.shape, generator=g).to(base)
    if kind == "all":
        return noise
    c = base.clone()                       # every 17th pixel changes
    c.view(-1, 3)[t % 17::17] = noise.view(-1, 3)[t % 17::17]
    return c


def _run(entry, bias, w, h, k, kind, n, r2k=None):
    over = dict(fovea_radius_px=0.05 * w + 1.0, seed=synth.PHILOX_SEED, stream_id=5, bias_mode=bias,
                **({} if r2k is None else {"r2k": r2k}))
    flags = fwrs.FLAG_REPROJECT if entry == "reproject" else 0
    res = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over, flags=flags), stream=torch.cuda.current_stream())
    orc = oracle.Oracle(w, h, k, oracle.default_params(w, **over))
    out = torch.full((h, w, 3), -1.0, device="cuda")
    spec = synth.StreamSpec(w, h, k, n, 0.05 * w + 1.0, 0.125 * w + 2.0, 2.0, 2, 6.0)
    src = synth.FrameSource(spec, device="cuda")
    moving = synth.MovingSource(spec, device="cuda", n_frames=n) if entry == "reproject" else None
    fov = fwrs.Foveator(w, h, 0.05 * w + 1.0, 0.125 * w + 2.0, fwrs.FOV_MIP,
                        stream=torch.cuda.current_stream()) if entry == "foveated" else None
    base = src.frame(0)[0].contiguous()
    entries = []
    for t in range(n):
        _, lev, gx, gy = src.frame(t)
        c = _colours(base, t, kind)
        if entry == "reproject":
            _, _, mv, d, _, _ = moving.frame(t)
            res.step_reproject(c, lev, mv, d, gx, gy, DEPTH_TOL, out)
            orc.push_reproject(c.cpu().numpy(), lev.cpu().numpy(), mv.cpu().numpy(), d.cpu().numpy(), gx, gy, DEPTH_TOL)
            continue
        if entry == "foveated":
            res.step_foveated(fov, c, gx, gy, out)
            orc.push(*oracle.foveate(c.cpu().numpy(), gx, gy, 0.05 * w + 1.0, 0.125 * w + 2.0, fwrs.FOV_MIP), gx, gy)
            continue
        orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
        if entry == "push":
            res.push(c, lev, gx, gy)
        elif entry == "step" or (entry == "incremental" and t == 0):
            res.step(c, lev, gx, gy, out)
        elif entry == "incremental":
            res.step_incremental(c, lev, gx, gy, out)
        else:
            entries.append((res, c, lev, gx, gy, out))
            if entry == "tick" or len(entries) == 2 or t == n - 1:
                fwrs.tick(entries)
                entries = []
    if entry == "push":
        res.resolve(out)
    res.sync()
    st, so = res.download(), orc.state()
    for name in ("cnt", "idx"):
        np.testing.assert_array_equal(getattr(st, name), getattr(so, name), err_msg=name)
    for name in ("wt", "col", "wslot"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32), err_msg=name)
    assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL


@pytest.mark.parametrize("entry", ["step", "push", "incremental", "tick", "group", "foveated", "reproject"])
@pytest.mark.parametrize("bias,kind", [(fwrs.BIAS_FULL, "all"), (fwrs.BIAS_FULL, "some"), (fwrs.BIAS_FULL, "still"),
                                       (fwrs.AES, "all")])
@pytest.mark.parametrize("w,h,k", [(65, 17, 1), (67, 9, 2), (63, 21, 3), (70, 13, 4), (61, 11, 5), (66, 10, 7),
                                   (62, 9, 8), (33, 9, 16)])
def test_every_pass(entry, bias, kind, w, h, k):
    _run(entry, bias, w, h, k, kind, 5)


@pytest.mark.parametrize("entry", ["step", "foveated"])
@pytest.mark.parametrize("k", [3, 5])
def test_untame_at_the_added_slot_counts(entry, k):
    _run(entry, fwrs.BIAS_FULL, 63, 21, k, "all", 5, r2k=1e-6)


@pytest.mark.parametrize("entry,bias,w,h,k", [
    ("push", fwrs.BIAS_FULL, 1920, 1460, 4), ("incremental", fwrs.BIAS_FULL, 1200, 1166, 8),
    ("foveated", fwrs.BIAS_FULL, 1920, 1460, 4), ("step", fwrs.AES, 1600, 1170, 6), ("tick", fwrs.BIAS_FULL, 1920, 1460, 4)])
def test_stores_above_the_cache(entry, bias, w, h, k):
    _run(entry, bias, w, h, k, "some", 2)
