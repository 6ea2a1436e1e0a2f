"""Deterministic 64-tap filtering of sorted streams (blocks that stage their tap
box in LDS beside blocks that sum by four lanes or a lane a query from global
memory) where texels are infinite or not numbers, the domain ends inside a leaf
along every axis, and leaves are missing: the results of the unsorted kernel,
bit for bit (not-a-number where that has it), scattered and in order."""
import numpy as np
import pytest
import torch

import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("fmt", ["f32", "f16", "bf16", "fp8_e4m3", "u8"])
@pytest.mark.parametrize("dims", [(48, 40, 56), (45, 37, 51)])
def test_sorted_streams_equal_unsorted_ones(dev, dims, fmt, special):
    if special and fmt == "u8":
        pytest.skip("8-bit codes are all finite")
    rng = np.random.default_rng(sum(dims))
    nb = [(d + 7) // 8 for d in dims]
    org = np.stack(np.meshgrid(*[np.arange(n) for n in nb], indexing="ij"), -1).reshape(-1, 3)
    org = (8 * org[rng.random(org.shape[0]) < 0.7]).astype(np.int32)
    vals = rng.random((org.shape[0], 8, 8, 8)).astype(np.float32)
    if special:
        hit = rng.random(vals.shape) < 0.002
        vals[hit] = rng.choice(np.array([np.nan] if fmt == "fp8_e4m3" else [np.nan, np.inf, -np.inf], np.float32), int(hit.sum()))
    tex = stf.stf_create_sparse_grid3d(dims, stf.FORMATS[fmt], org, synth.encode(vals, fmt), background=0.375)
    dense = synth.uniform_box_queries((12, 10, 14), 20000, seed=3) + np.float32(9.0)   # blocks that stage
    wide = synth.uniform_box_queries(dims, 6000, seed=4, margin=5.0)                   # blocks that do not
    p = np.concatenate([dense, wide, wide[:9] + np.float32(400.0)]).astype(np.float32)
    p[::501] = np.inf
    p = p[rng.permutation(p.shape[0])]
    q = torch.from_numpy(p).to(dev)
    n = p.shape[0]
    sq, order = torch.empty_like(q), torch.empty(n, dtype=torch.int32, device=dev)
    ws = torch.empty(stf.stf_sort_workspace_bytes(n), dtype=torch.uint8, device=dev)
    stf.stf_sort_queries(tex, q, sq, order, ws)
    for filt in (stf.STF_CUBIC_BSPLINE, stf.STF_CUBIC_KEYS):
        want = torch.empty((n, 1), device=dev)
        stf.stf_filter(tex, q, filt, stf.STF_DETERMINISTIC, 0, want)
        for flags, ref in ((stf.STF_ORDER_SCATTER, want), (0, want[order.long()])):
            got = torch.empty((n, 1), device=dev)
            stf.stf_stage_counting(True)
            stf.stf_filter_ordered(tex, sq, order, filt, stf.STF_DETERMINISTIC, 0, got, flags=flags)
            staged, blocks = stf.stf_stage_counts()
            stf.stf_stage_counting(False)
            assert 0 < staged < blocks, (staged, blocks)
            nan = torch.isnan(ref)
            assert torch.equal(torch.isnan(got), nan)
            assert torch.equal(got[~nan].view(torch.int32), ref[~nan].view(torch.int32)), (filt, flags)
    tex.destroy()
