"""Advantage estimation: results written over the inputs."""
import numpy as np
import pytest
import torch

from gpu_util import dev

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


@pytest.mark.parametrize("T,N", [(1, 3), (24, 65), (32, 64), (33, 130), (48, 4097), (100, 63), (7, 65537), (41, 66000), (5, 196609)])
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
