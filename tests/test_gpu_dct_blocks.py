"""Deterministic filtering of DCT textures by blocks (weight sums per axis and
block instead of a decode per tap) against the FP64 oracle, at the sizes where
the block split can go wrong: textures of one block, windows clamped at every
side, channel counts that end inside a group of four words, and Gaussian
windows that cover the whole texture.

Tolerance, relative to sum |w| A (A the sum of the magnitudes of a texel's six
terms): a channel accumulates m = 6 blocks terms and an axis nt weights, each
addition rounding once (at most 2^-24 of the scale, about 0.6 of that RMS), so
the sum is within 3 sqrt(m + 2 nt) 2^-24 (five standard deviations) plus 4
roundings of the factors."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth
from test_gpu_dct import FILTERS, _abs_terms, _texture

pytestmark = pytest.mark.gpu


def _tol(taps, blocks):
    return (4 + 3 * math.sqrt(6 * blocks + 2 * taps)) * 2.0 ** -24


def _uv(n, seed):
    uv = synth.uv_queries(n, seed=seed) * np.float32(1.6) - np.float32(0.3)   # a third outside the texture
    uv[:5] = [[np.nan, 0.5], [0.5, np.inf], [-40.0, 0.5], [0.5, 90.0], [1.0, 0.0]]
    return uv.astype(np.float32)


def _check(got, ref, scale, tol, what):
    err = np.abs(got.astype(np.float64) - ref)
    ok = (np.isnan(got) & np.isnan(ref)) | (err <= tol * scale)
    assert ok.all(), (what, int((~ok).sum()), float(np.nanmax(err / np.maximum(scale, 1e-30))), tol)


@pytest.mark.parametrize("W,H,C", [(8, 8, 1), (16, 8, 2), (8, 24, 4), (24, 16, 5), (40, 32, 9), (16, 16, 13)])
def test_dct_blocks_match_oracle(dev, W, H, C):
    words = stf.stf_dct_encode(_texture(H, W, C, seed=W + H + C))
    t = stf.stf_create_dct_texture2d(W, H, C, words)
    A = _abs_terms(words).astype(np.float32)
    uv = _uv(3001, W + C)   # the last block of the launch is partial
    q = torch.from_numpy(uv).to(dev)
    for fname, gf, of in FILTERS:
        gd = stf.filter(t, q, gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()
        od, _ = oracle.dct_filter2d(words, uv, of, oracle.DET)
        scale, _ = oracle.filter2d(A, oracle.F32, uv, of, oracle.DET_ABS)
        _check(gd, od, scale, _tol(2 if fname == "linear" else 4, 4), (fname, W, H, C))
    out = torch.empty((uv.shape[0], C), dtype=torch.float32, device=dev)
    for sigma in (0.2, 0.8, 4.0):
        sigma = float(np.float32(sigma))
        nt = 2 * math.ceil(6 * sigma) + 4
        for gm, om, taps in ((stf.STF_GAUSS_DISCRETE_MEAN, oracle.G_DISCRETE_MEAN, 4),
                             (stf.STF_GAUSS_FIS_MEAN, oracle.G_FIS_MEAN, nt)):
            stf.stf_filter_gaussian(t, q, sigma, gm, 0, out)
            od, _ = oracle.dct_gauss_filter2d(words, uv, sigma, om)
            scale, _ = oracle.gauss_filter2d(A, oracle.F32, uv, sigma, om)
            _check(out.cpu().numpy(), od, scale, _tol(taps, ((taps + 6) // 8 + 1) ** 2), (gm, sigma, W, H, C))
    t.destroy()
