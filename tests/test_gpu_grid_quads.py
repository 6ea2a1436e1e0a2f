"""Deterministic 64-tap filtering of grids where four lanes sum a query: waves
with every number of live queries (groups of 16 of them are summed together),
queries that repeat a cell (then a lane sums its own) beside scattered ones,
domains that end inside a leaf, missing leaves with a non-zero background, and
special values beside the taps.  Bar: 1e-6 of sum |w t| against the FP64
oracle; and the bits of a query do not depend on the queries beside it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

KINDS = [(stf.STF_CUBIC_BSPLINE, oracle.CUBIC), (stf.STF_CUBIC_MITCHELL, oracle.MITCHELL)]
OFMT = {"f32": oracle.F32, "f16": oracle.F16, "bf16": oracle.BF16, "fp8_e4m3": oracle.FP8_E4M3, "u8": oracle.U8}


def _grid(fmt, dims, seed, keep=0.6):
    rng = np.random.default_rng(seed)
    nb = [(d + 7) // 8 for d in dims]
    org = np.stack(np.meshgrid(*[np.arange(n) for n in nb], indexing="ij"), -1).reshape(-1, 3)
    org = org[rng.random(org.shape[0]) < keep]
    vals = rng.random((org.shape[0], 8, 8, 8)).astype(np.float32)
    return (8 * org).astype(np.int32), synth.encode(vals, fmt)


@pytest.mark.parametrize("fmt", list(OFMT))
@pytest.mark.parametrize("dims", [(32, 24, 40), (29, 21, 37)])
def test_quads_match_oracle(dev, fmt, dims):
    org, raw = _grid(fmt, dims, seed=sum(dims))
    bg = 0.375
    tex = stf.stf_create_sparse_grid3d(dims, stf.FORMATS[fmt], org, raw, background=bg)
    og = oracle.Grid(dims, OFMT[fmt], org, raw, bg)
    rng = np.random.default_rng(7)
    p = synth.uniform_box_queries(dims, 64 * 70 + 13, seed=8, margin=3.0)
    far = np.array([200.0, -90.0, 0.5], np.float32)   # no leaf, no tap
    for k in range(64):      # wave k: k + 1 queries near leaves, the rest far outside
        p[64 * k + rng.permutation(64)[:63 - k]] = far
    p[64 * 64:64 * 66] = p[64 * 64] + rng.random((128, 3), dtype=np.float32) * np.float32(0.3)   # one cell
    p[64 * 66:64 * 67:2] = p[64 * 66]                                                            # every other lane alike
    p[64 * 68 + 5] = [np.nan, 1, 1]
    p = p.astype(np.float32)
    q = torch.from_numpy(p).to(dev)
    perm = rng.permutation(p.shape[0])
    for gf, of in KINDS:
        got = stf.filter(tex, q, gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()[:, 0]
        ref, _ = og.filter(p, of, oracle.DET, 0)
        scale, _ = og.filter(p, of, oracle.DET_ABS, 0)
        ok = (np.isnan(got) & np.isnan(ref)) | (np.abs(got.astype(np.float64) - ref) <= 1e-6 * scale)
        assert ok.all(), (fmt, dims, gf, int((~ok).sum()))
        again = stf.filter(tex, torch.from_numpy(p[perm]).to(dev), gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()[:, 0]
        assert np.array_equal(again.view(np.uint32), got[perm].view(np.uint32))
    tex.destroy()


def test_special_values_reach_only_their_taps(dev):
    dims = (32, 24, 40)
    org, raw = _grid("f32", dims, seed=4)
    raw = raw.copy()
    raw[3, 4, 4, 4], raw[5, 0, 7, 0], raw[6] = np.inf, np.nan, 0.0
    raw[0, 0, 0, 0] = -np.inf   # the first stored voxel, which lanes without a chunk read
    tex = stf.stf_create_sparse_grid3d(dims, stf.STF_FMT_F32, org, raw)
    og = oracle.Grid(dims, oracle.F32, org, raw)
    p = synth.uniform_box_queries(dims, 20000, seed=9, margin=2.0)
    for gf, of in KINDS:
        got = stf.filter(tex, torch.from_numpy(p).to(dev), gf, stf.STF_DETERMINISTIC, 0)[0].cpu().numpy()[:, 0]
        ref, _ = og.filter(p, of, oracle.DET, 0)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    tex.destroy()
