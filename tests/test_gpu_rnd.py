"""RND reward at embedding widths and row counts around the edges of its kernels, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import assert_elementwise, dev, host, rel_l2
from oracle import rnd as ornd
from workloads import xavier_mlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _check(rx, K, N):
    g = np.random.default_rng(1000 * K + N)
    dims = (8, 16, K)
    pt, pp = xavier_mlp(g, dims), xavier_mlp(g, dims)
    obs, rew = g.normal(size=(N, 8)).astype(np.float32), g.normal(size=N).astype(np.float32)
    start = (0.4, 0.05, 1000.0)
    targ, pred = rx.Mlp(dims, dev(pt)), rx.Mlp(dims, dev(pp))
    running, d_rew, r_int = dev(np.array(start, np.float32)), dev(rew), torch.empty(N, device="cuda")
    ws = rx.workspace(rx.rslx_rnd_workspace_bytes(targ, N))
    rx.rslx_trace_begin(64)
    rx.rslx_rnd(targ, pred, dev(obs), N, 8, None, 8, running, 0.5, 1, r_int, d_rew, ws)
    torch.cuda.synchronize()
    sites = [r[0] for r in rx.rslx_trace_end()]
    ri_ref, _, run_ref = ornd.intrinsic_reward(pp, pt, dims, obs, start)
    # the bounds of test_rnd_reward
    assert rel_l2(host(r_int), ri_ref) < 1e-4
    assert_elementwise("r_int", host(r_int), ri_ref)
    np.testing.assert_allclose(host(d_rew), rew + 0.5 * ri_ref, rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(host(running), np.array(run_ref), rtol=1e-4)
    return sites


@pytest.mark.parametrize("K,N", [(64, 262144), (64, 262145)])
def test_long_lists_of_block_sums_are_folded_once(rx, K, N):
    """Above 4096 block sums of 64 rows one workgroup adds them up before all others read the result."""
    fold = ["rnd_fold"] if N > 4096 * 64 else []
    assert [n for n in _check(rx, K, N) if n.startswith("rnd")] == ["rnd_raw"] + fold + ["rnd_apply"]


@pytest.mark.parametrize("K,N", [(1, 1), (1, 257), (3, 255), (4, 256), (5, 65), (7, 300), (8, 257), (16, 63), (17, 65), (30, 65), (64, 64), (100, 130), (130, 129)])
def test_rnd_widths(rx, K, N):
    """Rows of one lane, of four and of sixteen, in 16-byte pieces or single columns, in one pass over the row or several."""
    _check(rx, K, N)
