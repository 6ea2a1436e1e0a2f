"""Rounding of the deterministic filters of DCT textures: weighing blocks has to
be at least as near to the FP64 oracle as the plain way, which decodes every
tap in binary32 and sums rows, then the column, in binary32 (emulated here).

Both errors are root mean squares over 80,000 values relative to the values'
own, so their spread between inputs is below a percent.  Emulated in binary32,
the ratio of the two lies between 0.56 and 0.86 (wide Gaussian windows); a DC
factor with the scale and the separately summed weights in it gives 1.0 to
1.85."""
import math

import numpy as np
import pytest
import torch
from scipy.special import erfc

import oracle
import paper_2305_05810_amd as stf
import synth
from test_gpu_dct import _texture

pytestmark = pytest.mark.gpu

f32 = np.float32
SIZE, CH, N = 256, 4, 20000
K, K11 = f32((2 / 15) / (4 * math.sqrt(2))), f32((2 / 15) / 4)
C1 = np.array([math.cos((2 * i + 1) * math.pi / 16) for i in range(8)]).astype(f32)
C2 = np.array([math.cos((2 * i + 1) * math.pi / 8) for i in range(8)]).astype(f32)


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(f32)


def _texels(words):
    """Every texel decoded in binary32: (H, W, C)."""
    w = np.repeat(np.repeat(words, 8, 0), 8, 1)
    x1, x2 = (np.tile(t, SIZE // 8)[None, :, None] for t in (C1, C2))
    y1, y2 = (np.tile(t, SIZE // 8)[:, None, None] for t in (C1, C2))
    f = (w & 127).astype(f32) * f32(1 / 127)
    for k, b in enumerate((K * x1, K * y1, K * y2, (K11 * x1) * y1, K * x2)):
        f = _fma(((w >> (7 + 5 * k)) & 31).astype(f32) - f32(16), b, f)
    return f


def _weights(kind, t):
    """Scaled binary32 weights of one axis, their scale, offset of the first tap."""
    one, s = f32(1), f32(1) - t
    if kind == "linear":
        return [s, t], 1, 0
    if kind == "bspline":
        st = s * t
        return [s * s * s, one + (3 * s) * (one + st), one + (3 * t) * (one + st), t * t * t], 6, -1
    if kind == "keys":
        return [-((t * s) * s), s * (2 + t * (2 - 3 * t)), t * (2 + s * (2 - 3 * s)), -((t * t) * s)], 2, -1
    if kind == "mitchell":
        m = f32(-7)
        return [(s * s) * _fma(m, t, one), one + s * (9 + s * (27 - 21 * s)), one + t * (9 + t * (27 - 21 * t)),
                (t * t) * _fma(m, s, one)], 18, -1
    sigma, t = kind[1], t.astype(np.float64)
    if kind[0] == "discrete_mean":
        w = [np.exp(-(k - t) ** 2 / (2 * sigma * sigma)) for k in range(-1, 3)]
        return [(v / sum(w)).astype(f32) for v in w], 1, -1
    r = math.ceil(6 * sigma) + 1
    edge = [0.5 * erfc(-(k - 0.5 - t) / sigma / math.sqrt(2)) for k in range(-r, r + 3)]
    return [(b - a).astype(f32) for a, b in zip(edge, edge[1:])], 1, -r


def _plain(texels, uv, kind):
    x, y = uv[:, 0] * f32(SIZE) - f32(0.5), uv[:, 1] * f32(SIZE) - f32(0.5)
    cx, cy = np.floor(x).astype(int), np.floor(y).astype(int)
    wx, scale, o = _weights(kind, x - cx.astype(f32))
    wy, _, _ = _weights(kind, y - cy.astype(f32))
    acc = np.zeros((len(uv), CH), f32)
    for j, b in enumerate(wy):
        row = np.zeros((len(uv), CH), f32)
        for i, a in enumerate(wx):
            row = _fma(a[:, None], texels[np.clip(cy + o + j, 0, SIZE - 1), np.clip(cx + o + i, 0, SIZE - 1)], row)
        acc = _fma(b[:, None], row, acc)
    return acc / f32(scale * scale)


KINDS = ["linear", "bspline", "keys", "mitchell", ("discrete_mean", 0.5), ("fis_mean", 0.5), ("fis_mean", 2.0)]


@pytest.mark.parametrize("codes", ["encoded", "random"])
@pytest.mark.parametrize("kind", KINDS, ids=str)
def test_dct_blocks_round_no_worse_than_taps(dev, kind, codes):
    if codes == "encoded":
        words = stf.stf_dct_encode(_texture(SIZE, SIZE, CH, seed=31))
    else:
        rng = np.random.default_rng(32)
        words = rng.integers(0, 128, (SIZE // 8, SIZE // 8, CH)).astype(np.uint32)
        for k in range(5):
            words |= rng.integers(1, 32, words.shape).astype(np.uint32) << np.uint32(7 + 5 * k)
    uv = synth.uv_queries(N, seed=33)
    t = stf.stf_create_dct_texture2d(SIZE, SIZE, CH, words)
    q = torch.from_numpy(uv).to(dev)
    if isinstance(kind, str):
        f, of = {"linear": (stf.STF_LINEAR, oracle.LINEAR), "bspline": (stf.STF_CUBIC_BSPLINE, oracle.CUBIC),
                 "keys": (stf.STF_CUBIC_KEYS, oracle.KEYS), "mitchell": (stf.STF_CUBIC_MITCHELL, oracle.MITCHELL)}[kind]
        got = stf.filter(t, q, f, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()
        exact, _ = oracle.dct_filter2d(words, uv, of, oracle.DET)
    else:
        g, og = {"discrete_mean": (stf.STF_GAUSS_DISCRETE_MEAN, oracle.G_DISCRETE_MEAN),
                 "fis_mean": (stf.STF_GAUSS_FIS_MEAN, oracle.G_FIS_MEAN)}[kind[0]]
        out = torch.empty((N, CH), dtype=torch.float32, device=dev)
        stf.stf_filter_gaussian(t, q, kind[1], g, 0, out)
        got = out.cpu().numpy()
        exact, _ = oracle.dct_gauss_filter2d(words, uv, kind[1], og)
    t.destroy()
    plain = _plain(_texels(words), uv, kind)
    mine, theirs = (float(np.sqrt(np.mean((v.astype(np.float64) - exact) ** 2))) for v in (got, plain))
    assert theirs < 1e-6 * float(np.sqrt(np.mean(exact ** 2)))   # the emulation filters the same texture
    assert mine <= theirs, (kind, codes, mine / theirs)
