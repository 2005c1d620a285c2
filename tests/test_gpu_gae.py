"""Advantage estimation: chunk edges and kernel choice against the oracle, results written over the inputs."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host
from oracle import gae as ogae

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _inputs(T, N, seed):
    g = np.random.default_rng(seed)
    timeouts = (g.random((T, N)) < 0.05).astype(np.uint8)
    return dict(rewards=g.normal(size=(T, N)).astype(np.float32), values=g.normal(size=(T, N)).astype(np.float32),
                last=g.normal(size=N).astype(np.float32), dones=(g.random((T, N)) < 0.05).astype(np.uint8) | timeouts, timeouts=timeouts)


@pytest.mark.parametrize("T,N", [(1, 3), (24, 65), (32, 64), (33, 130), (48, 4097), (100, 63), (7, 65537), (41, 66000), (5, 196609), (5, 393217)])
def test_gae_in_place(rx, T, N):
    """Advantages over the rewards and returns over the values, and the other way round: the bits of separate buffers."""
    d = {k: dev(v) for k, v in _inputs(T, N, T + N).items()}
    ws = rx.workspace(rx.rslx_gae_workspace_bytes(T, N))
    for normalize in (False, T * N > 1):
        call = lambda r, v, a, q: rx.rslx_gae(r, v, d["last"], d["dones"], d["timeouts"], T, N, 0.99, 0.95, normalize, a, q, ws)  # noqa: E731
        adv, ret = torch.empty(T, N, device="cuda"), torch.empty(T, N, device="cuda")
        call(d["rewards"], d["values"], adv, ret)
        r, v = d["rewards"].clone(), d["values"].clone()
        call(r, v, r, v)
        assert torch.equal(r, adv) and torch.equal(v, ret), normalize
        r, v = d["rewards"].clone(), d["values"].clone()
        call(r, v, v, r)
        assert torch.equal(v, adv) and torch.equal(r, ret), normalize


@pytest.mark.parametrize("T,N", [(31, 64), (32, 65), (33, 64), (48, 100), (64, 1), (65, 333), (100, 1), (8, 16384), (24, 16385), (9, 40001),
                                 (24, 65535), (3, 196607), (3, 196608), (3, 393215), (3, 393216)])
@pytest.mark.parametrize("timeouts", [False, True])
def test_gae_sizes(rx, T, N, timeouts):
    i = _inputs(T, N, 7 * T + N)
    d = {k: dev(v) for k, v in i.items()}
    adv, ret = torch.empty(T, N, device="cuda"), torch.empty(T, N, device="cuda")
    ws = rx.workspace(rx.rslx_gae_workspace_bytes(T, N))
    a_ref, r_ref = ogae.gae(i["rewards"], i["values"], i["last"], i["dones"], 0.99, 0.95, timeouts=i["timeouts"] if timeouts else None)
    rx.rslx_trace_begin(4)
    for normalize in (False, True):
        rx.rslx_gae(d["rewards"], d["values"], d["last"], d["dones"], d["timeouts"] if timeouts else None, T, N, 0.99, 0.95, normalize, adv, ret, ws)
        torch.cuda.synchronize()
        ref = ogae.normalize_advantages(a_ref) if normalize else a_ref
        # T fused multiply-adds per column, each of 2^-24 of a running value that gamma lambda keeps within about 20 terms
        assert np.max(np.abs(host(ret) - r_ref)) <= 1e-5 * max(1.0, np.max(np.abs(r_ref)))
        assert np.max(np.abs(host(adv) - ref)) <= 2e-5 * max(1.0, np.max(np.abs(ref)))
    # eight wavefronts per 64 columns while every CU has one workgroup of it, one lane per column above
    site = "gae_scan" if N <= 16384 else "gae_columns"
    assert [r[0] for r in rx.rslx_trace_end()] == [site, site + "+normalize"]
