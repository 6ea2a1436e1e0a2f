"""Shading by a lane per column of the window (two or four lanes a query):
batches that end inside a wave and a block, windows that cross every border of
a level that is no multiple of the 4 x 4 tiles, coordinates outside it, and
directions below the horizon, opposite (no half vector) or not finite, where
the unlit taps give zero.  Against the oracle, with the bounds of
test_gpu_shade.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

SHADE_REL, SHADE_ABS = 1e-4, 1e-6


@pytest.mark.parametrize("size,levels", [(1, 1), (5, 1), (6, 2), (12, 3), (64, 3)])
@pytest.mark.parametrize("fname", ["linear", "cubic"])
def test_ends_borders_and_directions(dev, size, levels, fname):
    lv = synth.material_levels(size, seed=size, levels=levels)
    mat = stf.stf_create_material2d(size, size, lv)
    ref = oracle.Material(lv)
    recs = synth.shade_queries(1100, seed=size + 1)
    rng = np.random.default_rng(size)
    recs[:, :2] = rng.uniform(-0.4, 1.4, (1100, 2))
    recs[::50, 0] = np.nan
    recs[7::50, 1] = -np.inf
    recs[3::40, 6:9] = -recs[3::40, 3:6]        # opposite: no half vector
    recs[9::40, 5] = -recs[9::40, 5]            # below the horizon
    recs[13::40, 8] = -recs[13::40, 8]
    recs[17::80, 4] = np.nan                    # a direction that is not one: no tap is lit
    q = torch.from_numpy(recs).to(dev)
    filt, of = (stf.STF_LINEAR, oracle.LINEAR) if fname == "linear" else (stf.STF_CUBIC_BSPLINE, oracle.CUBIC)
    for gm, om in ((stf.STF_SHADE_AFTER_FILTER, oracle.SH_AFTER_FILTER), (stf.STF_FILTER_AFTER_SHADE, oracle.SH_FILTER_AFTER),
                   (stf.STF_SHADE_STOCHASTIC, oracle.SH_STOCH)):
        want, _ = ref.shade(recs, of, om, 3)
        for n in (1, 15, 16, 17, 63, 64, 65, 127, 129, 255, 257, 1100):
            out = torch.full((n + 1, 3), -3.0, device=dev)
            stf.stf_shade_filter(mat, q[:n], filt, gm, 3, out[:n])
            g = out.cpu().numpy().astype(np.float64)
            assert np.all(g[n] == -3.0)
            g, o = g[:n], want[:n]
            ok = (np.isnan(g) & np.isnan(o)) | (np.abs(g - o) <= SHADE_REL * np.abs(o) + SHADE_ABS)
            assert ok.all(), (gm, n, np.argwhere(~ok)[:4], g[~ok][:4], o[~ok][:4])
    mat.destroy()
