"""Requests in flight together whose queries and results are on either side
(those with results on the device share their round's event, the others have
one each): every request's results equal the same lookups filtered alone, with
rounds of many requests and of few; a cancelled request ends done or cancelled
and the server goes on.  A replay's requests that are due together are
submitted, waited for and released in groups of 256."""
import numpy as np
import pytest
import torch

import paper_2305_05810_amd as stf
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tex():
    g = synth.fbm_grid((64, 64, 64), base_period=16.0, seed=7)
    return g, stf.stf_create_sparse_grid3d(g.dims, stf.STF_FMT_F32, g.origins, g.values)


def _alone(tex, q, seed):
    return stf.filter(tex, q, stf.STF_CUBIC_BSPLINE, stf.STF_STOCHASTIC, seed, want_index=True)


@pytest.mark.parametrize("max_resident,chunk", [(1, 100), (3, 64), (64, 1000)])
def test_either_side(dev, tex, max_resident, chunk):
    g, t3 = tex
    srv = stf.stf_server_create(8 << 20, max_resident, chunk)
    rng = np.random.default_rng(max_resident)
    sent = []
    for k in range(40):
        q = synth.uniform_box_queries(g.dims, int(rng.integers(1, 700)), seed=k, margin=2.0)
        qd = torch.from_numpy(q).to(dev)
        ref, ridx = _alone(t3, qd, k)
        if k % 2:
            out, idx = torch.empty_like(ref), torch.empty_like(ridx)
        else:
            out, idx = np.empty(tuple(ref.shape), np.float32), np.empty(tuple(ridx.shape), np.int32)
        torch.cuda.synchronize()
        sent.append((stf.stf_server_submit(srv, t3, qd if k // 2 % 2 else q, stf.STF_CUBIC_BSPLINE, k, out, idx), out,
                     idx, ref, ridx))
    stf.stf_server_cancel(srv, sent[-1][0])
    for k, (t, out, idx, ref, ridx) in enumerate(sent):
        try:
            stf.stf_server_wait(srv, t)
        except stf.STFError:
            assert k == len(sent) - 1
        else:
            assert np.array_equal(torch.as_tensor(out).cpu().numpy(), ref.cpu().numpy())
            assert np.array_equal(torch.as_tensor(idx).cpu().numpy(), ridx.cpu().numpy())
        stf.stf_server_release(srv, t)
    st = stf.stf_server_stats(srv)
    assert st["completed"] + st["cancelled"] == 40 and st["resident"] == 0 and st["pending"] == 0
    srv.destroy()


@pytest.mark.parametrize("count", [1, 256, 257, 600])
def test_replay_of_a_burst(dev, tex, count):
    g, t3 = tex
    srv = stf.stf_server_create(8 << 20, 300, 64)
    n = 130
    q = torch.from_numpy(synth.uniform_box_queries(g.dims, n * count, seed=count, margin=2.0)).to(dev)
    out = torch.full((n * count, 1), -3.0, device=dev)
    reqs = [(t3, q.data_ptr() + 12 * n * k, n, stf.STF_CUBIC_BSPLINE, k, out.data_ptr() + 4 * n * k, None,
             0.0 if k < count - 5 else 0.002) for k in range(count)]
    torch.cuda.synchronize()
    for _ in range(2):
        out.fill_(-3.0)
        torch.cuda.synchronize()
        stf.stf_server_replay(srv, reqs, stf.STF_SERVE_QUERIES_ON_DEVICE | stf.STF_SERVE_RESULTS_ON_DEVICE, 30.0)
        for k in range(0, count, 37):
            assert torch.equal(out[n * k:n * (k + 1)], _alone(t3, q[n * k:n * (k + 1)], k)[0].reshape(n, 1))
        assert not (out == -3.0).any()
    st = stf.stf_server_stats(srv)
    assert st["completed"] == 2 * count and st["queries"] == 2 * count * n and st["resident"] == 0 and st["pending"] == 0
    srv.destroy()
