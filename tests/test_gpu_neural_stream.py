"""Adam steps of latents too large for the caches (their moments go past them):
two steps of the same samples, the second with the moments that the first one
left.  With latents stepped by lr0 = 0 no gradient changes between the steps, so
g, (m1, v1) and (m2, v2) are the formulas', and untouched latents stay."""
import numpy as np
import pytest
import torch

import paper_2305_05810_amd as stf
from test_gpu_neural_tiles import _pcg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("LW,LH", [(2048, 1024), (2048, 512)])   # 2^24 latent values and half of them
def test_second_step_has_the_first_ones_moments(dev, LW, LH):
    rng = np.random.default_rng(2)
    lat = rng.normal(0, 0.3, (LH, LW, 8)).astype(np.float32)
    mlp = rng.normal(0, 0.25, stf.stf_ntex_param_count()).astype(np.float32)
    nt = stf.stf_ntex_create(LW, LH, lat, mlp)
    tgt = torch.rand(LH, LW, 8, device=dev)
    B, seed = 64, 5
    g = []
    for step in (1, 2):
        key = int(_pcg(seed ^ int(_pcg(0))))
        h = _pcg(np.arange(B, dtype=np.uint64) ^ _pcg(key ^ step))
        pos = np.stack([h % LW, _pcg((h + np.uint64(1)) & np.uint64(0xFFFFFFFF)) % LH], axis=1).astype(np.int32)
        gl, gm = torch.empty((LH, LW, 8), device=dev), torch.empty(mlp.size, device=dev)
        stf.stf_ntex_gradients(nt, tgt, torch.from_numpy(pos).to(dev), gl, gm)
        g.append(gl.cpu().numpy().astype(np.float64))
        stf.stf_ntex_train(nt, tgt, 1, B, 0.0 if step == 1 else 1e-2, 0.0, seed)
    got, _ = stf.stf_ntex_get_params(nt)
    nt.destroy()
    m = 0.9 * (0.1 * g[0]) + 0.1 * g[1]
    v = 0.999 * (0.001 * g[0] ** 2) + 0.001 * g[1] ** 2
    want = (m / (1 - 0.9 ** 2)) / (np.sqrt(v / (1 - 0.999 ** 2)) + 1e-8)
    step = (lat.astype(np.float64) - got) / 1e-2
    hit = (g[0] != 0) | (g[1] != 0)
    assert hit.any() and np.array_equal(got[~hit], lat[~hit])
    big = hit & (np.maximum(np.abs(g[0]), np.abs(g[1])) >= max(1e-4 * np.abs(g[0]).max(), 1e-6))
    assert np.all(np.abs(step - want)[big] < 1e-3 + 2.0 ** -22 * np.abs(lat[big]) / 1e-2)
