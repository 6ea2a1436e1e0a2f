"""Deterministic 64-tap filtering of unsorted grid queries at the batch sizes
where the division of a call changes (queries a wave, four lanes a query or a
lane each): a query has the same bits in every batch, and those within 1e-6 of
sum |w t| of the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

LINES = [24576, 65536, 98304, 131072, 262144]


@pytest.mark.parametrize("fmt,ofmt", [("f32", oracle.F32), ("f16", oracle.F16), ("u8", oracle.U8)])
def test_a_query_has_its_bits_in_every_batch(dev, fmt, ofmt):
    dims = (61, 40, 53)
    rng = np.random.default_rng(5)
    nb = [(d + 7) // 8 for d in dims]
    org = np.stack(np.meshgrid(*[np.arange(n) for n in nb], indexing="ij"), -1).reshape(-1, 3)
    org = (8 * org[rng.random(org.shape[0]) < 0.6]).astype(np.int32)
    raw = synth.encode(rng.random((org.shape[0], 8, 8, 8)).astype(np.float32), fmt)
    tex = stf.stf_create_sparse_grid3d(dims, stf.FORMATS[fmt], org, raw, background=0.25)
    n = LINES[-1] + 70
    p = synth.uniform_box_queries(dims, n, seed=9, margin=4.0)
    walk = np.arange(n) // 200 % 2 == 0        # every second run of 200 steps through the box in small steps
    p[walk] = p[np.arange(n) // 200 * 200][walk] + (np.arange(n) % 200)[walk, None] * np.float32(0.11)
    far = np.arange(n) // 500 % 5 == 4
    p[far] += np.float32(500.0)
    p[::701] = np.nan
    q = torch.from_numpy(p.astype(np.float32)).to(dev)
    whole = torch.empty((n, 1), device=dev)
    stf.stf_filter(tex, q, stf.STF_CUBIC_BSPLINE, stf.STF_DETERMINISTIC, 0, whole)
    ids = rng.choice(n, 3000, replace=False)
    og = oracle.Grid(dims, ofmt, org, raw, 0.25)
    want, _ = og.filter(p[ids].astype(np.float32), oracle.CUBIC, oracle.DET)
    scale, _ = og.filter(p[ids].astype(np.float32), oracle.CUBIC, oracle.DET_ABS)
    got = whole.cpu().numpy()[ids, 0]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    fin = ~np.isnan(want)
    assert np.all(np.abs(got[fin] - want[fin]) <= 1e-6 * scale[fin])
    for m in [1, 31, 32, 33, 127, 128, 129] + [k + d for k in LINES for d in (0, 1)]:
        out = torch.full((m + 1, 1), -3.0, device=dev)
        stf.stf_filter(tex, q[:m], stf.STF_CUBIC_BSPLINE, stf.STF_DETERMINISTIC, 0, out[:m])
        assert torch.equal(out[:m].view(torch.int32), whole[:m].view(torch.int32)), m
        assert out[m].item() == -3.0
    tex.destroy()
