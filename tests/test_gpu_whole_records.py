"""The passes that read every record -- contexts without a resolve plane, the first frames of a session, the
resolve alone -- at the edges of their tiles and lane groups: widths and heights that cut tiles short, every
group size, frames in which few or all pixels replace slots, tame and untame."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2510_03964_amd import fwrs, synth

pytestmark = pytest.mark.gpu
COLOR_TOL = 1e-5     # binary32 weighted mean of at most 16 values in [0, 1] against binary64


@pytest.mark.parametrize("entry", ["step", "push+resolve", "tick"])
@pytest.mark.parametrize("w,h,k,tile", [(64, 4, 1, None), (65, 5, 1, (8, 8)), (63, 3, 2, None), (130, 67, 2, (32, 8)),
                                        (67, 41, 3, (16, 4)), (129, 65, 4, None), (131, 9, 4, (8, 32)), (1, 1, 4, None),
                                        (66, 33, 5, None), (130, 64, 8, (64, 2)), (63, 65, 8, None), (63, 33, 16, None)])
@pytest.mark.parametrize("r2k", [None, 1e-6])
def test_every_record_read(entry, w, h, k, tile, r2k):
    n = 9
    spec = synth.StreamSpec(w, h, k, n, max(1.0, 0.05 * w), max(2.0, 0.125 * w), 2.0, 2, 6.0)
    src = synth.FrameSource(spec, device="cuda")
    over = dict(fovea_radius_px=spec.fovea_radius_px, seed=synth.PHILOX_SEED, **({} if r2k is None else {"r2k": r2k}))
    res = fwrs.Reservoir(w, h, k, fwrs.default_params(w, **over, flags=fwrs.FLAG_NO_RESOLVE_PLANE),
                         stream=torch.cuda.current_stream())
    if tile:
        res.set_tile(*tile)
    orc = oracle.Oracle(w, h, k, oracle.default_params(w, **over))
    out = torch.full((h, w, 3), -1.0, device="cuda")
    for t in range(n):
        c, lev, gx, gy = src.frame(t)
        if entry == "step":
            res.step(c, lev, gx, gy, out)
        elif entry == "tick":
            fwrs.tick([(res, c, lev, gx, gy, out)])
        else:
            res.push(c, lev, gx, gy)
            res.resolve(out)
        orc.push(c.cpu().numpy(), lev.cpu().numpy(), gx, gy)
        assert np.abs(out.cpu().numpy().astype(np.float64) - orc.resolve()).max() <= COLOR_TOL
    st, so = res.download(), orc.state()
    np.testing.assert_array_equal(st.idx, so.idx)
    for name in ("wsum", "wt", "col"):
        np.testing.assert_array_equal(getattr(st, name).view(np.uint32), getattr(so, name).view(np.uint32))
    takes, changed, updates = res.stats()
    assert updates == n * w * h and w * h <= changed <= takes
