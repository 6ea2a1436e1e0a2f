"""Bilinear filtering of DCT textures at the batch size where a call goes from a
thread per query and group of four channels to a thread per query: a query has
the same bits in every batch, ordered and scattered ones too, and those of the
FP64 oracle within the bound of test_gpu_dct_blocks.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
from test_gpu_dct import _abs_terms, _texture
from test_gpu_dct_blocks import _check, _tol, _uv

pytestmark = pytest.mark.gpu

LINE = 65536


@pytest.mark.parametrize("W,H,C", [(8, 8, 5), (64, 24, 8), (40, 32, 9), (16, 16, 13), (48, 8, 16)])
def test_a_query_has_its_bits_in_every_batch(dev, W, H, C):
    words = stf.stf_dct_encode(_texture(H, W, C, seed=W + C))
    t = stf.stf_create_dct_texture2d(W, H, C, words)
    n = LINE + 300
    uv = _uv(n, W + H)
    q = torch.from_numpy(uv).to(dev)
    whole = torch.empty((n, C), device=dev)
    stf.stf_filter(t, q, stf.STF_LINEAR, stf.STF_DETERMINISTIC, 0, whole)
    od, _ = oracle.dct_filter2d(words, uv, oracle.LINEAR, oracle.DET)
    scale, _ = oracle.filter2d(_abs_terms(words).astype(np.float32), oracle.F32, uv, oracle.LINEAR, oracle.DET_ABS)
    _check(whole.cpu().numpy(), od, scale, _tol(2, 4), (W, H, C))
    for m in (1, 2, 63, 64, 65, 255, 257, 3001, LINE - 1, LINE, LINE + 1):
        out = torch.full((m + 1, C), -3.0, device=dev)
        stf.stf_filter(t, q[:m], stf.STF_LINEAR, stf.STF_DETERMINISTIC, 0, out[:m])
        assert torch.equal(out[:m].view(torch.int32), whole[:m].view(torch.int32)), m
        assert bool((out[m] == -3.0).all())
    m = 3001
    sq, order = torch.empty_like(q[:m]), torch.empty(m, dtype=torch.int32, device=dev)
    ws = torch.empty(stf.stf_sort_workspace_bytes(m), dtype=torch.uint8, device=dev)
    stf.stf_sort_queries(t, q[:m].contiguous(), sq, order, ws)
    for flags, ref in ((stf.STF_ORDER_SCATTER, whole[:m]), (0, whole[:m][order.long()])):
        out = torch.empty((m, C), device=dev)
        stf.stf_filter_ordered(t, sq, order, stf.STF_LINEAR, stf.STF_DETERMINISTIC, 0, out, flags=flags)
        assert torch.equal(out.view(torch.int32), ref.contiguous().view(torch.int32)), flags
    t.destroy()
