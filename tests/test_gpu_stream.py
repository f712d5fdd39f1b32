"""The passes that work through a list of pixels, at the edges of their launch rules: two tiles per wave from
4096 work items on (fwrs_push_frame and the incremental call), widths that cut tiles and groups of lanes short,
and every group size (1, 2, 4, 8 and 16 lanes per pixel, whole and partly used)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2510_03964_amd import fwrs, synth

pytestmark = pytest.mark.gpu
COLOR_TOL = 1e-5     # binary32 weighted mean of at most 16 values in [0, 1] against binary64


@pytest.mark.parametrize("entry", ["incremental", "push"])
@pytest.mark.parametrize("w,h,k", [(1024, 1023, 4), (1024, 1024, 4), (1001, 1030, 3), (1023, 1025, 16),
                                   (1025, 1024, 1), (1090, 997, 8), (1024, 1025, 2), (1100, 960, 6)])
def test_two_tiles_per_wave(entry, w, h, k):
    spec = synth.StreamSpec(w, h, k, 5, 0.05 * w, 0.125 * w, 2.0, 2, 6.0)
    src = synth.FrameSource(spec, device="cuda")
    over = dict(fovea_radius_px=spec.fovea_radius_px, seed=synth.PHILOX_SEED)
    res = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over), stream=torch.cuda.current_stream())
    orc = oracle.Oracle(w, h, k, oracle.default_params(w, **over))
    out = torch.full((h, w, 3), -1.0, device="cuda")
    for t in range(spec.frames):
        c, lev, gx, gy = src.frame(t)
        if entry == "push":
            res.push(c, lev, gx, gy)
        elif t == 0:
            res.step(c, lev, gx, gy, out)
        else:
            res.step_incremental(c, lev, gx, gy, out)
        orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
    if entry == "push":
        res.resolve(out)
    st, so = res.download(), orc.state()
    np.testing.assert_array_equal(st.idx, so.idx)
    for name in ("wsum", "wt", "col"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32))
    assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL
    takes, changed, updates = res.stats()
    assert updates == spec.frames * w * h and w * h <= changed <= takes


@pytest.mark.parametrize("bias", [fwrs.BIAS_FULL, fwrs.AES])
@pytest.mark.parametrize("entry", ["step", "push", "incremental", "tick"])
@pytest.mark.parametrize("w,h,k", [(130, 67, 1), (131, 66, 2), (67, 41, 4), (129, 65, 5), (130, 64, 8), (63, 33, 16),
                                   (1200, 1165, 8), (1200, 1166, 8)])
def test_per_slot_modes_by_slot_count_and_store_size(bias, entry, w, h, k):
    """One lane per slot or per pixel (k = 4, 8), and stores on either side of the size from which the records
    are streamed (1200 x 1165.08 at k = 8)."""
    big = w * h > 1 << 20
    if big and (entry != "step" or bias == fwrs.AES):
        pytest.skip("the size rule is the same for every entry point")
    spec = synth.StreamSpec(w, h, k, 3 if big else 6, 0.05 * w, 0.125 * w, 2.0, 2, 6.0)
    src = synth.FrameSource(spec, device="cuda")
    over = dict(fovea_radius_px=spec.fovea_radius_px, seed=synth.PHILOX_SEED, bias_mode=bias)
    res = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over), stream=torch.cuda.current_stream())
    orc = oracle.Oracle(w, h, k, oracle.default_params(w, **over))
    out = torch.full((h, w, 3), -1.0, device="cuda")
    for t in range(spec.frames):
        c, lev, gx, gy = src.frame(t)
        if entry == "push":
            res.push(c, lev, gx, gy)
        elif entry == "tick":
            fwrs.tick([(res, c, lev, gx, gy, out)])
        elif entry == "step" or t == 0:
            res.step(c, lev, gx, gy, out)
        else:
            res.step_incremental(c, lev, gx, gy, out)
        orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
    if entry == "push":
        res.resolve(out)
    st, so = res.download(), orc.state()
    np.testing.assert_array_equal(st.idx, so.idx)
    for name in ("wt", "col", "wslot"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32))
    assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL
    takes, changed, updates = res.stats()
    assert updates == spec.frames * w * h and w * h <= changed <= takes
