"""How a call's decodes are spread over pairs of batches and waves does not
change a result: with 4 queries a pair (16 taps), 16 (4 taps) or 64 (one tap)
and one pair a turn up to 3072 pairs, two beyond, the first queries of a call
equal those of a shorter one bit for bit, and a deterministic result follows
its query to any place of the batch.  Sides and latent ratios differ per axis,
and non-finite coordinates stay in their own query's result.  A sample is
checked against the oracle that rounds at the same points."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu

W, H, LW, LH = 96, 40, 24, 20
INFER_ABS = 1e-2   # one bfloat16 ulp of a hidden activation moves an output by less (see test_gpu_neural.py)


@pytest.fixture(scope="module")
def nt(dev):
    rng = np.random.default_rng(7)
    lat = (rng.standard_normal((LH, LW, 8)) * 0.5).astype(np.float32)
    _, mlp = synth.neural_init(16, seed=3)
    mlp = (mlp + 0.05 * rng.standard_normal(mlp.shape)).astype(np.float32)   # biases too
    t = stf.stf_ntex_create(W, H, lat, mlp)
    stf.stf_ntex_prepare_inference(t)
    yield t, lat, mlp
    t.destroy()


def _run(t, q, filt, mode):
    out = torch.full((q.shape[0], 8), -5.0, device=q.device)
    stf.stf_ntex_filter(t, q, filt, mode, 11, out)
    return out


@pytest.mark.parametrize("mode", ["deterministic", "stochastic"])
@pytest.mark.parametrize("fname", ["linear", "cubic"])
def test_results_do_not_depend_on_the_split(dev, nt, fname, mode):
    t, lat, mlp = nt
    filt = stf.STF_LINEAR if fname == "linear" else stf.STF_CUBIC_BSPLINE
    md = stf.STF_DETERMINISTIC if mode == "deterministic" else stf.STF_STOCHASTIC
    per = 64 if mode == "stochastic" else (16 if fname == "linear" else 4)
    edge = 3072 * per
    n = 2 * edge + per + 1
    rng = np.random.default_rng(n)
    uv = rng.uniform(-0.1, 1.1, (n, 2)).astype(np.float32)
    bad = rng.integers(0, n, 40)
    uv[bad[:20], 0] = np.nan
    uv[bad[20:], 1] = np.inf
    q = torch.from_numpy(uv).to(dev)
    full = _run(t, q, filt, md)
    fin = np.isfinite(uv).all(1)
    assert np.array_equal(torch.isfinite(full).all(1).cpu().numpy(), fin)
    assert np.array_equal(torch.isnan(full).all(1).cpu().numpy(), ~fin)
    for m in (1, per - 1, per, per + 1, 2 * per + 1, 5 * per, edge - 1, edge, edge + 1, edge + per + 1, 2 * edge):
        assert torch.equal(_run(t, q[:m].contiguous(), filt, md).nan_to_num(-7), full[:m].nan_to_num(-7)), m
    if mode == "deterministic":
        for s in (1, 3, per + 2):
            rolled = _run(t, torch.roll(q, s, 0), filt, md)
            assert torch.equal(rolled.nan_to_num(-7), torch.roll(full, s, 0).nan_to_num(-7)), s
    on = oracle.NeuralTexture(lat.astype(np.float16).astype(np.float64), mlp, W, H)
    ref, _ = on.filter(uv[:512], oracle.LINEAR if fname == "linear" else oracle.CUBIC,
                       oracle.DET if mode == "deterministic" else oracle.STOCH, seed=11, emulate=True)
    err = np.abs(full[:512].cpu().numpy().astype(np.float64) - ref)[fin[:512]]
    assert err.max() < INFER_ABS
