"""Deterministic 2D filtering where rows of taps are read whole: widths around
a row (below it every tap is loaded by itself) and around a wave, waves wholly
inside the texture, waves with lanes at and beyond every border, partial waves,
every storage format and channel count, and special values beside the taps.  Bar: 1e-6 of sum |w t| against the FP64 oracle (the
repository's bar for deterministic filters)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

FMTS = {"f32": oracle.F32, "f16": oracle.F16, "bf16": oracle.BF16, "fp8_e4m3": oracle.FP8_E4M3, "u8": oracle.U8}
FILTERS = [(stf.STF_LINEAR, oracle.LINEAR), (stf.STF_CUBIC_BSPLINE, oracle.CUBIC), (stf.STF_CUBIC_KEYS, oracle.KEYS)]


def _queries(W, H, n):
    """First half inside (x and y at least 3 texels from every border), then
    uniform over the texture and beyond."""
    rng = np.random.default_rng(W + H)
    uv = rng.random((n, 2)) * 1.2 - 0.1
    h = n // 2 // 64 * 64
    uv[:h] = (np.array([3.0, 3.0]) + rng.random((h, 2)) * np.array([max(W - 6.0, 0.0), max(H - 6.0, 0.0)])) / np.array([W, H])
    uv = uv.astype(np.float32)
    uv[-3:] = [[np.nan, 0.5], [0.5, np.inf], [-3.0, 4.0]]
    return uv


@pytest.mark.parametrize("fmt", list(FMTS))
@pytest.mark.parametrize("W,H,C", [(64, 9, 1), (65, 8, 2), (67, 30, 3), (64, 64, 4), (63, 20, 4), (200, 3, 1), (1, 5, 3),
                                   (2, 2, 4), (3, 9, 1), (4, 4, 2), (5, 1, 3), (6, 7, 1)])
def test_rows_match_oracle(dev, fmt, W, H, C):
    t = synth.texture2d(W, H, C, seed=W * C)
    raw = synth.encode(t, fmt)
    tex = stf.stf_create_texture2d(W, H, C, stf.FORMATS[fmt], [raw])
    uv = _queries(W, H, 1001)
    q = torch.from_numpy(uv).to(dev)
    for gf, of in FILTERS:
        got = stf.filter(tex, q, gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy().astype(np.float64)
        ref, _ = oracle.filter2d(raw.reshape(H, W, C), FMTS[fmt], uv, of, oracle.DET)
        scale, _ = oracle.filter2d(raw.reshape(H, W, C), FMTS[fmt], uv, of, oracle.DET_ABS)
        ok = (np.isnan(got) & np.isnan(ref)) | (np.abs(got - ref) <= 1e-6 * scale)
        assert ok.all(), (fmt, W, H, C, gf, int((~ok).sum()))
    tex.destroy()


@pytest.mark.parametrize("W", [64, 23])
def test_special_values_reach_only_their_taps(dev, W):
    H = 16
    t = synth.texture2d(W, H, 2, seed=3)
    t[5, 20], t[6, 21, 0], t[0, 0], t[H - 1, W - 1] = np.inf, np.nan, -np.inf, np.nan
    tex = stf.stf_create_texture2d(W, H, 2, stf.STF_FMT_F32, [t])
    uv = _queries(W, H, 4096)
    for gf, of in FILTERS:
        got = stf.filter(tex, torch.from_numpy(uv).to(dev), gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()
        ref, _ = oracle.filter2d(t, oracle.F32, uv, of, oracle.DET)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    tex.destroy()
