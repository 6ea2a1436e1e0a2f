"""16-tap decoding of a neural texture at the batch sizes where the division of a
call among the waves changes (one pair of batches a wave, up to two resident
sets of them, then two pairs a turn): a query has the same bits in every call
(the values themselves are held to the oracle by test_gpu_neural.py and
test_gpu_neural_pairs.py)."""
import numpy as np
import pytest
import torch

import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

SET = 3072 * 4   # queries of one resident set, a pair of batches (four queries) a wave


@pytest.mark.parametrize("mode", [stf.STF_DETERMINISTIC, stf.STF_STOCHASTIC])
@pytest.mark.parametrize("filt", [stf.STF_LINEAR, stf.STF_CUBIC_BSPLINE])
def test_a_query_has_its_bits_in_every_call(dev, filt, mode):
    rng = np.random.default_rng(8)
    lat = (rng.standard_normal((16, 16, 8)) * 0.3).astype(np.float32)
    mlp = (rng.standard_normal(stf.stf_ntex_param_count()) * 0.2).astype(np.float32)
    nt = stf.stf_ntex_create(64, 64, lat, mlp)
    stf.stf_ntex_prepare_inference(nt)
    n = 4 * SET + 7
    uv = synth.uv_queries(n, seed=3) * np.float32(1.4) - np.float32(0.2)
    uv[::97, 0] = np.nan
    q = torch.from_numpy(uv.astype(np.float32)).to(dev)
    whole = torch.empty((n, 8), device=dev)
    stf.stf_ntex_filter(nt, q, filt, mode, 11, whole)
    bad = torch.isnan(q).any(1)
    assert bool(torch.isnan(whole[bad]).all()) and not bool(torch.isnan(whole[~bad]).any())
    for m in (1, 3, 4, 5, 64, 65, SET - 1, SET, SET + 1, 2 * SET - 3, 2 * SET, 2 * SET + 1, 2 * SET + 5, 3 * SET):
        out = torch.full((m + 1, 8), -3.0, device=dev)
        stf.stf_ntex_filter(nt, q[:m], filt, mode, 11, out[:m])
        assert torch.equal(out[:m].view(torch.int32), whole[:m].view(torch.int32)), m
        assert bool((out[m] == -3.0).all())
    stf.stf_ntex_destroy(nt)
