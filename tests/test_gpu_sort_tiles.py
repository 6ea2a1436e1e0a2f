"""Tile sizes of the radix sort: a tile is 1024, 2048 or 4096 keys by the
batch's size.  The order is the stable argsort of the Morton keys at the edges
of a tile, of the digit table's lines (16 tiles) and of the rule's bands; a
workspace that holds a batch holds every smaller one."""
import numpy as np
import pytest
import torch

import paper_2305_05810_amd as stf
import synth

BAND8, BAND16 = 3 << 19, 3 << 20


def test_workspace_never_shrinks_with_the_batch():
    edges = [1, 1024, 1025, 16 * 1024, 17 * 1024 + 1, 1 << 20, BAND8 - 1, BAND8, BAND8 + 1, 2 << 20, BAND16 - 1, BAND16,
             BAND16 + 1, 6 << 20, 6 << 20 | 1, 1 << 24, (1 << 31) - 1]
    sizes = [stf.stf_sort_workspace_bytes(n) for n in edges]
    assert sizes == sorted(sizes)
    assert all(b >= 16 * n for n, b in zip(edges, sizes))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 15 * 1024 + 1, 16 * 1024, 33 * 1024 + 7, BAND8 - 1, BAND8,
                               BAND8 + 2049, BAND16 - 1, BAND16, BAND16 + 4097])
@pytest.mark.parametrize("kind", ["grid", "2d"])
def test_order_at_tile_edges(dev, n, kind):
    rng = np.random.default_rng(n)
    if kind == "grid":
        g = synth.fbm_grid((64, 48, 40), base_period=16.0, seed=5)
        tex = stf.stf_create_sparse_grid3d(g.dims, stf.STF_FMT_F32, g.origins, g.values)
        q = rng.uniform(-3.0, 67.0, (n, 3)).astype(np.float32)
        dims, shift = (64, 48, 40), 3
        c = np.floor(q).astype(np.int64) >> shift
    else:
        tex = stf.stf_create_texture2d(200, 37, 1, stf.STF_FMT_F32, [rng.random((37, 200), dtype=np.float32)])
        q = rng.uniform(-0.05, 1.05, (n, 2)).astype(np.float32)
        dims, shift = (200, 37), 2
        c = np.floor(q * np.float32(dims) - np.float32(0.5)).astype(np.int64) >> shift
    cells = [(d + (1 << shift) - 1) >> shift for d in dims]
    bits = (max(cells) - 1).bit_length()
    key = np.zeros(n, np.int64)
    for a, m in enumerate(cells):
        v = np.clip(c[:, a], 0, m - 1)
        for b in range(bits):
            key |= ((v >> b) & 1) << (len(dims) * b + a)
    bad = rng.integers(0, n, size=min(n // 8, 5))
    q[bad] = np.nan
    key[bad] = 1 << (len(dims) * bits)
    want = np.argsort(key, kind="stable")
    sq, order = stf.sort_queries(tex, torch.from_numpy(q).to(dev))
    assert np.array_equal(order.cpu().numpy(), want)
    assert np.array_equal(sq.cpu().numpy().view(np.uint32), q[want].view(np.uint32))
